// Device code of the sparse-weight-sync hot path for gfx950 (wave64, 256 CUs in 8 XCDs).
//
// extract_kernel: one pass over old/new.  Each workgroup is assigned a bucket by its block id
//   (consecutive block ids rotate over a group of buckets, so that many buckets are in flight at
//   once) and claims that bucket's next tile with an atomic ticket on the bucket's own counter:
//   tickets on one address serialise at about 11 ns each on this chip, spread over 32 addresses
//   they cost nothing.  A tile is a run of up to TILE = 2048*V elements inside one tensor and one
//   bucket.  Ticket order within a bucket is start order, which is what makes the chained scan
//   free of deadlock whatever order the hardware dispatches workgroups in.  The workgroup streams
//   both inputs with 16-byte loads, forms per-lane change masks by XOR of the 16-bit patterns
//   (Alg. 1: I = { i : W[i] != W_prev[i] }), ranks the changed elements with a packed DPP wave
//   scan + an LDS combine across the four waves, chains tiles of the same bucket with a
//   decoupled look-back on one 64-bit {flag, value} status word per tile, stages the
//   (index, value) pairs of the tile in LDS in rank order and writes them out coalesced, by one wave once the others are done
//   (Alg. 2: V = W[I], I int32 ascending).  The snapshot is refreshed in the same pass: 128-byte lines of
//   it that hold a change are rewritten from the new weights the lanes hold (RG = 8), or each changed
//   element is stored by itself (RG = 0), or nothing is written for callers that rotate buffers (RG = -1).
//   Template flavours of the same kernel: SRC = FP32 master weights rounded to BF16 on the fly (the
//   cast-and-copy of Alg. 1 fused with its diff); EB = 1 for one-byte (FP8) patterns.
// mark_kernel: one optimizer step of Alg. 1's index accumulation, OR-ed into a bitmap.
// extract_marked_kernel: the payload of the accumulated index set, gathered through the bitmap.
// apply_kernel: the scatter of Alg. 3, W[I] <- V, one workgroup per (bucket, payload chunk);
//   apply_grouped_kernel: the same where the payload slots hold whole buckets, several chunks per workgroup.
// refresh_overflow_kernel: whole-bucket copy for buckets whose payload overflowed, when the snapshot is refreshed
// by scattering the payload into it after the scan (apply_kernel on the snapshot) instead of inside extract_kernel.
// apply_encoded_kernel / encode_indices_kernel: the 16-bit index delta coding of Sec. 3.3.
// route_kernel / dense_copy_kernel: the per-bucket sparse / dense routing of Sec. 3.4 and its full-copy route.
//
// No arithmetic is done on weight values anywhere (the cast flavour rounds, nothing more); every kernel here
// is HBM-bandwidth bound and there is no contraction, hence no MFMA.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <stdint.h>

namespace srs {

constexpr int kThreads = 256;          // 4 waves of 64
constexpr int kWaves = kThreads / 64;
constexpr int kVecElems = 8;           // 16-byte vector = 8 patterns
constexpr int kUnit = kThreads * kVecElems;   // 2048 elements per "V" step of a tile
constexpr uint32_t kStage = 2048;      // (index,value) pairs staged in LDS per round
constexpr uint32_t kApplyChunk = 2048; // payload pairs per apply workgroup
constexpr int kLoadPace = 4;           // s_sleep argument between the streaming loads of an extract that refreshes in place

constexpr uint32_t kFlagOverflow = 1u, kFlagBadIndex = 2u, kFlagTimeout = 4u;
constexpr uint32_t kFlagsReported = 7u;
constexpr uint32_t kFlagStatic = 1u << 31;     // with kFlagTimeout: raised by a launch on the library's static scratch; not reported
constexpr uint32_t kStAgg = 1u, kStPrefix = 2u;   // tile status: aggregate only / inclusive prefix

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Weight pointers reach the kernels through tables in device memory, so the compiler cannot tell that they are
// global addresses and would use FLAT loads and stores for them (which also occupy the LDS queue and the LDS
// counter).  Every such pointer is cast to the global address space once, where it is read from its table:
// the streaming loads then compile to global_load_dwordx4 and measure 3 % faster on the 910-bucket benchmark set.
#define SRS_GLOBAL __attribute__((address_space(1)))
template <class T> using gptr = T SRS_GLOBAL *;
template <class T> __device__ __forceinline__ gptr<T> as_global(T *p) { return (gptr<T>)p; }
// a uniform pointer that stays in scalar registers: the accesses of a lane then share one offset register, instead of each having
// a 64-bit address of its own
template <class T> __device__ __forceinline__ gptr<T> scalar_base(gptr<T> p) {
    uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(unsigned long long)p);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((unsigned long long)p >> 32));
    asm("" : "+s"(lo), "+s"(hi));
    return (gptr<T>)(((unsigned long long)hi << 32) | lo);
}

struct TileDesc {          // one extract tile of a tensor list (16 bytes)
    uint32_t tensor;       // index into the pointer table
    uint32_t tensor_off;   // first element inside the tensor
    uint32_t bucket_off;   // first element inside the bucket
    uint32_t len;          // 1 .. TILE
};

struct WgInfo {            // what one extract workgroup serves (16 bytes)
    uint32_t bucket;       // the bucket whose next tile it claims
    uint32_t first_tile;   // id of that bucket's first tile
    uint32_t ntiles;       // number of tiles of that bucket
    uint32_t pad;
};

struct SegDesc {           // a run of one tensor inside one bucket (16 bytes)
    uint32_t bucket_off;
    uint32_t len;
    uint32_t tensor;
    uint32_t tensor_off;
};

struct PtrPair { uint16_t *old_w; const void *new_w; };   // new_w: BF16 weights, or FP32 master weights (CAST)

struct ExtractArgs {
    // single tensor: nb buckets of tiles_per_bucket tiles each, the last one of last_tiles tiles
    uint16_t *old_w; const void *new_w; uint64_t n; uint32_t be; uint32_t tiles_per_bucket;
    uint32_t nb; uint32_t last_tiles; uint32_t group;      // group = buckets interleaved per group
    // tensor list
    const TileDesc *tiles; const PtrPair *ptrs;
    const WgInfo *wg_info;          // [ntiles] bucket served by each workgroup
    const uint32_t *bucket_first;   // [nb+1] id of each bucket's first tile
    uint32_t ntiles;
    int32_t *I; uint16_t *V; uint32_t *counts; uint64_t cap;
    unsigned long long *status;     // [status_cap >= ntiles] {epoch, flag : value}
    uint64_t status_cap;
    uint32_t *tickets;              // per-bucket ticket counters, ticket_stride words apart, all 0 between launches
    uint32_t ticket_stride;
    uint32_t *epoch;                // epoch[0]: this launch's epoch; epoch[kEpochClaimed]: buckets whose tickets are all taken
    uint32_t chained;               // buckets of more than one tile
    uint32_t *flags;
    uint32_t timeout;               // what a tile that gives up raises in them
    uint32_t spin_limit;
    // cumulative changed-index set: one bit per packed position (bit g&31 of word g>>5)
    uint32_t *bitmap; uint64_t bitmap_words; const uint64_t *tensor_base;   // packed position of each tensor's element 0
};

struct ApplyArgs {
    // single tensor
    uint16_t *w; uint64_t n;
    // tensor list
    const SegDesc *segs; const uint32_t *seg_begin; uint16_t *const *wptrs; uint64_t total;
    uint32_t be; uint32_t nb; uint32_t chunks_per_bucket;
    const int32_t *I; const uint16_t *V; const uint32_t *counts; uint64_t cap;
    uint32_t *flags;
    // pointers to skip between two entries of wptrs: 0 for the apply-side table, 1 when wptrs is the extract-side
    // table of PtrPair read through its old_w members (the second-pass snapshot refresh)
    uint32_t wptr_skip;
    // apply_grouped_kernel: chunks of each bucket that have a workgroup of their own, chunks per workgroup behind them
    uint32_t direct, group;
    // 16-bit index coding (null / 0 for apply_kernel, whose payload carries 32-bit indices only)
    const uint16_t *D; const uint32_t *max_gap; const int32_t *anchors; uint64_t base_stride;
};

// ---------------------------------------------------------------------------------------------
// wave64 helpers
// ---------------------------------------------------------------------------------------------

template <int CTRL, int ROW_MASK, int BANK_MASK>
__device__ __forceinline__ uint32_t dpp_get(uint32_t x) {
    // lanes whose source is outside the row, or whose row is masked off, receive 0
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, BANK_MASK, ROW_MASK == 0xF && BANK_MASK == 0xF);
}

// inclusive prefix sum over the 64 lanes of a wave (also valid on two packed 16-bit fields as long
// as neither field overflows)
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
    x += dpp_get<0x111, 0xF, 0xF>(x);   // row_shr:1
    x += dpp_get<0x112, 0xF, 0xF>(x);   // row_shr:2
    x += dpp_get<0x114, 0xF, 0xF>(x);   // row_shr:4
    x += dpp_get<0x118, 0xF, 0xF>(x);   // row_shr:8
    x += dpp_get<0x142, 0xA, 0xF>(x);   // row_bcast:15 -> rows 1 and 3
    x += dpp_get<0x143, 0xC, 0xF>(x);   // row_bcast:31 -> rows 2 and 3
    return x;
}

// workgroup barrier that orders LDS accesses only: waits for this wave's LDS operations (lgkmcnt), not for its
// outstanding global loads and stores, before the barrier instruction
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");          // the compiler keeps LDS accesses on their side of it
    __builtin_amdgcn_s_waitcnt(0xC07F);     // vmcnt and expcnt at their maxima (= no wait), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ uint32_t lane63(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

__device__ __forceinline__ uint32_t uniform(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

template <bool NT>
__device__ __forceinline__ u32x4 load16(gptr<const void> p) {
    gptr<const u32x4> q = (gptr<const u32x4>)p;
    if (NT) return __builtin_nontemporal_load(q);
    return *q;
}
// the same at any address: one global_load_dwordx4 all the same (unaligned access is on for every HSA process)
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
template <bool NT>
__device__ __forceinline__ u32x4 load16_any(gptr<const void> p) {
    gptr<const u32x4_any> q = (gptr<const u32x4_any>)p;
    u32x4_any v;
    if (NT) v = __builtin_nontemporal_load(q);
    else v = *q;
    return (u32x4)v;
}
__device__ __forceinline__ void store16_nt(gptr<void> p, u32x4 v) { __builtin_nontemporal_store(v, (gptr<u32x4>)p); }

// binary32 pattern -> BF16 pattern, round to nearest even; NaN -> 0x7FC0
__device__ __forceinline__ uint32_t round_bf16(uint32_t x) {
    const uint32_t r = (x + 0x7FFFu + ((x >> 16) & 1u)) >> 16;
    return ((x & 0x7FFFFFFFu) > 0x7F800000u) ? 0x7FC0u : r;
}

// eight consecutive master weights (two 16-byte vectors) -> eight BF16 patterns in memory order
__device__ __forceinline__ u32x4 round8_bf16(u32x4 f0, u32x4 f1) {
    u32x4 r;
    r.x = round_bf16(f0.x) | (round_bf16(f0.y) << 16);
    r.y = round_bf16(f0.z) | (round_bf16(f0.w) << 16);
    r.z = round_bf16(f1.x) | (round_bf16(f1.y) << 16);
    r.w = round_bf16(f1.z) | (round_bf16(f1.w) << 16);
    return r;
}

// The elements lo .. hi-1 (of the vector's 8) at p, which may lie before the first element that exists; the others
// read as 0.
__device__ __forceinline__ u32x4 load8_window(gptr<const uint16_t> p, uint32_t lo, uint32_t hi) {
    uint32_t h[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) h[k] = (k >= lo && k < hi) ? (uint32_t)p[k] : 0u;
    u32x4 r;
    r.x = h[0] | (h[1] << 16); r.y = h[2] | (h[3] << 16);
    r.z = h[4] | (h[5] << 16); r.w = h[6] | (h[7] << 16);
    return r;
}
__device__ __forceinline__ u32x4 load8_window_cast(gptr<const uint32_t> p, uint32_t lo, uint32_t hi) {
    uint32_t h[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) h[k] = (k >= lo && k < hi) ? round_bf16(p[k]) : 0u;
    u32x4 r;
    r.x = h[0] | (h[1] << 16); r.y = h[2] | (h[3] << 16);
    r.z = h[4] | (h[5] << 16); r.w = h[6] | (h[7] << 16);
    return r;
}

// bit k of the result is set iff the k-th 16-bit pattern of a and b differ (k = 0..7, memory order)
__device__ __forceinline__ uint32_t diff_mask8(u32x4 a, u32x4 b) {
    uint32_t m = 0;
    const uint32_t d0 = a.x ^ b.x, d1 = a.y ^ b.y, d2 = a.z ^ b.z, d3 = a.w ^ b.w;
    m |= (d0 & 0xFFFFu) ? 1u : 0u;   m |= (d0 >> 16) ? 2u : 0u;
    m |= (d1 & 0xFFFFu) ? 4u : 0u;   m |= (d1 >> 16) ? 8u : 0u;
    m |= (d2 & 0xFFFFu) ? 16u : 0u;  m |= (d2 >> 16) ? 32u : 0u;
    m |= (d3 & 0xFFFFu) ? 64u : 0u;  m |= (d3 >> 16) ? 128u : 0u;
    return m;
}

__device__ __forceinline__ uint32_t pattern_at(u32x4 v, uint32_t e) {
    const uint32_t lo = (e & 2u) ? v.y : v.x;
    const uint32_t hi = (e & 2u) ? v.w : v.z;
    const uint32_t w = (e & 4u) ? hi : lo;
    return (e & 1u) ? (w >> 16) : (w & 0xFFFFu);
}

// 16 one-byte patterns: elements lo .. hi-1 at p, the others read as 0
__device__ __forceinline__ u32x4 load16_window_u8(gptr<const uint8_t> p, uint32_t lo, uint32_t hi) {
    uint32_t d[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        uint32_t w = 0;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) w |= ((4 * q + k >= lo && 4 * q + k < hi) ? (uint32_t)p[4 * q + k] : 0u) << (8 * k);
        d[q] = w;
    }
    u32x4 r;
    r.x = d[0]; r.y = d[1]; r.z = d[2]; r.w = d[3];
    return r;
}

// bit k of the result is set iff byte k of d is non-zero (k = 0..3)
__device__ __forceinline__ uint32_t nonzero_bytes4(uint32_t d) {
    const uint32_t t = ((d | ((d & 0x7F7F7F7Fu) + 0x7F7F7F7Fu)) & 0x80808080u) >> 7;   // bits 0, 8, 16, 24
    return (t * 0x10204080u) >> 28;                                                       // gathered into bits 0..3
}

// Element width.  EB = 2: BF16 / FP16 patterns, 8 per 16-byte vector; EB = 1: FP8 patterns, 16 per vector
// (Sec. 2.1 measures the changed-element density at all three synchronisation precisions; nothing in
// Alg. 1-3 depends on the width).  diff_mask has one bit per element of the vector, in memory order.
template <int EB> struct Elem;
template <> struct Elem<2> {
    typedef uint16_t type;
    static __device__ __forceinline__ uint32_t diff_mask(u32x4 a, u32x4 b) { return diff_mask8(a, b); }
    static __device__ __forceinline__ uint32_t pattern(u32x4 v, uint32_t e) { return pattern_at(v, e); }
    static __device__ __forceinline__ u32x4 load_window(gptr<const uint16_t> p, uint32_t lo, uint32_t hi) {
        return load8_window(p, lo, hi);
    }
};
template <> struct Elem<1> {
    typedef uint8_t type;
    static __device__ __forceinline__ uint32_t diff_mask(u32x4 a, u32x4 b) {
        return nonzero_bytes4(a.x ^ b.x) | (nonzero_bytes4(a.y ^ b.y) << 4) | (nonzero_bytes4(a.z ^ b.z) << 8) |
               (nonzero_bytes4(a.w ^ b.w) << 12);
    }
    static __device__ __forceinline__ uint32_t pattern(u32x4 v, uint32_t e) {
        const uint32_t lo = (e & 4u) ? v.y : v.x;
        const uint32_t hi = (e & 4u) ? v.w : v.z;
        const uint32_t w = (e & 8u) ? hi : lo;
        return (w >> ((e & 3u) * 8u)) & 0xFFu;
    }
    static __device__ __forceinline__ u32x4 load_window(gptr<const uint8_t> p, uint32_t lo, uint32_t hi) {
        return load16_window_u8(p, lo, hi);
    }
};

__device__ __forceinline__ unsigned long long status_load(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void status_store(unsigned long long *p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long status_word(uint32_t epoch, uint32_t flag, uint32_t value) {
    return ((unsigned long long)((epoch << 2) | flag) << 32) | value;
}
// what a status word says in this epoch: its flag, 0 where it was written in another one
__device__ __forceinline__ uint32_t status_flag(uint32_t epoch, unsigned long long w) {
    const uint32_t hi = (uint32_t)(w >> 32);
    return ((hi ^ (epoch << 2)) < 4u) ? (hi & 3u) : 0u;
}

// Tables that no kernel of the launch writes, read at uniform addresses: in the constant address space they come through the
// scalar cache wherever they are read; behind an atomic or a barrier the compiler would take vector loads.
template <class T> __device__ __forceinline__ const T __attribute__((address_space(4))) *as_table(const T *p) {
    return (const T __attribute__((address_space(4))) *)p;
}

template <bool SCALAR, class T> __device__ __forceinline__ auto table(const T *p) {
    if constexpr (SCALAR) return as_table(p);
    else return p;
}

// ---------------------------------------------------------------------------------------------
// Tickets and status words need no clearing between launches.  A ticket counter is incremented exactly once per tile
// of its bucket and wraps to 0 with the last (atomic increment with a limit); status words carry the epoch of the launch that
// wrote them, and those of other epochs count as not written.  The epoch is state of the device, so that a replayed
// graph gets a new one each time: a workgroup reads it before it takes its ticket; the one that takes a bucket's last
// ticket counts the bucket, and the one that counts the last bucket raises the epoch, when every workgroup of the
// launch has read it, whatever else becomes of them.  The 30 bits of an epoch in a status word come round after 2^30
// launches; nothing written so long ago is left then: the tiles of chains write their words in every launch, tiles alone in
// their buckets wipe theirs now and then, and the workgroup that raises the epoch wipes 64 words behind the launch's tiles, other
// ones each time.
// The kernel that cleared both ahead of each launch took 1.4 us where little else ran and 4.7 us in a busy stream, and the
// host 2.5 us.  Extract and apply with it / without, us: 64 K elements 13.7 / 11.0, 1 M in four buckets 13.5 / 12.1, 4 M in
// four 17.5 / 16.0, 300 odd-sized tensors 147.5 / 146.1.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kEpochClaimed = 16;     // words between the epoch and the count of claimed buckets

// this launch's epoch; to be called before claim_tile
__device__ __forceinline__ uint32_t launch_epoch(const ExtractArgs &a) {
    const uint32_t e = *as_table(a.epoch);
    asm volatile("" : : "s"(e) : "memory");                  // it is here before the ticket is asked for
    return e;
}
__device__ __forceinline__ uint32_t claim_tile(const ExtractArgs &a, uint32_t bucket, uint32_t ntiles) {
    return atomicInc(a.tickets + (uint64_t)bucket * a.ticket_stride, ntiles - 1u);
}
// One lane of the workgroup that holds the last ticket of a bucket counts it; the result goes to raise_epoch.
__device__ __forceinline__ uint32_t count_claimed(const ExtractArgs &a) {
    uint32_t zero = 0;
    asm volatile("" : "+v"(zero));           // not uniform to the compiler, which would otherwise wait for the result on the spot
    return atomicInc(a.epoch + kEpochClaimed + zero, a.chained - 1u);
}
// All lanes of that wave, any time later.
__device__ __forceinline__ void raise_epoch(const ExtractArgs &a, uint32_t epoch, uint32_t counted, int lane) {
    if (uniform(counted) != a.chained - 1u) return;
    if (lane == 0) __hip_atomic_store(a.epoch, epoch + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t slices = (a.status_cap + 63u) / 64u, w = (epoch % slices) * 64u + (uint64_t)lane;
    if (w >= a.ntiles && w < a.status_cap) status_store(a.status + w, 0ull);
}

// Epoch and flag that an earlier launch left in a tile's status word.  This one's epoch is among them only where the epoch was
// not raised since, because calls that share the counters overlapped: the words are no counts then, and publish says so.
// Only a bucket's first tile looks, which waits for nobody afterwards: free, where all tiles looking costs single tensors of
// up to 16 M elements 1 to 5 %.
__device__ __forceinline__ uint32_t left_behind(const ExtractArgs &a, uint32_t tile) {
    return as_table(reinterpret_cast<const uint32_t *>(a.status + tile))[1];
}
// One lane of a bucket's only tile, which has no use for its word: leaves 0 there in one launch of 2^14, other tiles each time.
// (In every launch that takes the marked extract of 600 tensors in buckets of 3000 elements 5 %.)
__device__ __forceinline__ void wipe_alone(const ExtractArgs &a, uint32_t tile) {
    if ((((tile >> 6) ^ *as_table(a.epoch)) & 0x3FFFu) == 0) status_store(a.status + tile, 0ull);
}
// One lane: the tile's count.  A bucket's last tile, whose word nobody reads, leaves 0 there.
__device__ __forceinline__ void publish(const ExtractArgs &a, uint32_t epoch, uint32_t tile, uint32_t found, bool first, bool last, uint32_t total) {
    if (status_flag(epoch, (unsigned long long)found << 32) != 0) atomicOr(a.flags, a.timeout);
    status_store(a.status + tile, last ? 0ull : status_word(epoch, first ? kStPrefix : kStAgg, total));
}

// ---------------------------------------------------------------------------------------------
// decoupled look-back, run by all 64 lanes of wave 0.  Returns the number of changed elements in
// the tiles first_tile .. tile-1 of the same bucket.  Lane l inspects tile (pos - l); the window
// slides back by 64 until a tile with an inclusive prefix, or the bucket's first tile, is reached.
// Bounded: after spin_limit polls of one window the wave gives up, raises kFlagTimeout and
// returns what it has (ranks are clamped by the caller, so memory safety does not depend on it).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t look_back(const ExtractArgs &a, uint32_t epoch, uint32_t tile, uint32_t first_tile, int lane) {
    uint32_t excl = 0;
    int64_t pos = (int64_t)tile - 1;
    while (pos >= (int64_t)first_tile) {
        const int64_t idx = pos - lane;
        const bool in_bucket = idx >= (int64_t)first_tile;
        uint32_t flag = 0, value = 0;
        unsigned long long need = 0;
        bool found_prefix = false;
        uint32_t polls = 0;
        for (;;) {
            if (in_bucket && flag == 0) {                                    // only lanes still waiting poll again
                const unsigned long long w = status_load(a.status + idx);
                flag = status_flag(epoch, w);
                value = (uint32_t)w;
            }
            const unsigned long long valid = __ballot(in_bucket);            // a low run of lanes
            const unsigned long long pending = __ballot(in_bucket && flag == 0);
            const unsigned long long prefixed = __ballot(in_bucket && flag == kStPrefix);
            found_prefix = prefixed != 0;
            if (found_prefix) {
                const int first = __builtin_ctzll(prefixed);                 // nearest tile that has a prefix
                need = (first == 63) ? ~0ull : ((1ull << (first + 1)) - 1ull);
            } else {
                need = valid;
            }
            if ((pending & need) == 0) break;
            if (++polls > a.spin_limit) {
                if (lane == 0) atomicOr(a.flags, a.timeout);
                need &= ~pending;
                found_prefix = true;                                         // stop walking back
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        const uint32_t mine = ((need >> lane) & 1ull) ? value : 0u;
        excl += lane63(wave_inclusive_scan(mine));
        if (found_prefix) break;
        pos -= 64;
    }
    return excl;
}

// Refresh by lines of a tile read on extract_kernel's grid (og: grid position 0, g0: this lane's first, m: change
// masks, x: what to write): 8 consecutive grid vectors from a 128-byte boundary on, which begins q lanes before lane 0's
// vector; the line across the end of a row has its other vectors in the next row.
template <int V, class T>
__device__ __forceinline__ void refresh_lines(gptr<T> og, uint32_t g0, uint32_t nbody, bool in_head, const uint32_t (&m)[V],
                                              const u32x4 (&x)[V], int lane) {
    constexpr uint32_t ROW = 64u * 16u / sizeof(T);
    const uint32_t q = ((uint32_t)(uintptr_t)og >> 4) & 7u;             // uniform
    if (q == 0) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const unsigned long long changed = __ballot(m[j] != 0);
            const uint32_t g = g0 + j * ROW;
            if (((uint32_t)(changed >> (lane & ~7)) & 0xFFu) && g < nbody && (j > 0 || !in_head)) store16_nt(og + g, x[j]);
        }
    } else {
        const int first = (int)(((uint32_t)lane + q) & ~7u) - (int)q;                            // -7 .. 63
        unsigned long long prev = 0, cur = __ballot(m[0] != 0);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const unsigned long long next = (j + 1 < V) ? __ballot(m[(j + 1) % V] != 0) : 0ull;
            uint32_t line = (first < 0) ? (uint32_t)((cur << -first) | (prev >> (64 + first))) : (uint32_t)(cur >> first);
            if (first > 56) line |= (uint32_t)(next << (64 - first));
            const uint32_t g = g0 + j * ROW;
            if ((line & 0xFFu) && g < nbody && (j > 0 || !in_head)) store16_nt(og + g, x[j]);
            prev = cur; cur = next;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// extract
// ---------------------------------------------------------------------------------------------
// RG = how the snapshot is refreshed.  8: by whole lines -- the tile rewrites each
// aligned 128-byte line of the snapshot that holds a change (8 lanes x 16 bytes) from the
// new weights it has in registers; unchanged elements get the value they already hold.  (A wave rewrites its part of a line
// that reaches beyond its part of the tile if that part holds a change; the incomplete vectors go element by element.)  The snapshot's loads and
// these stores carry the non-temporal hint: a line written in full needs no read-modify-write behind the L2, and
// nothing of the snapshot is needed again.  Measured on the 910-bucket benchmark set against element-wise refresh,
// in one process, ms: 21.8 / 22.4 at 0.1 % changed, 25.8 / 28.7 at 1 %, 30.1 / 36.2 at 3 %, 33.6 / 40.4 at 10 %.
// The two hints only pay together (at 1 %: stores alone 27.6, loads alone 28.3; 64-byte blocks 28.8, 256-byte
// blocks 30.5).  The new weights are hinted as well (read once; worth 1 % on one-byte and on sparse data, nothing
// at 1 %), except the FP32 master weights of CAST, where the hint costs 1 ms of 38.
// 0: element by element everywhere (2-byte stores from the write-out loop).  -1: the snapshot is not touched at all
// (the caller rotates buffers: `new` is the next call's `old`).
// CAST: `new` is not a BF16 buffer but the FP32 master weights; each element is rounded to BF16
// (nearest even, NaN -> 0x7FC0) on the fly and `old` is the model-parameter buffer itself: the cast-and-
// copy of Alg. 1 fused with its diff, so that no snapshot exists at all.
// (The cumulative index set of Alg. 1 has a kernel of its own, extract_marked_kernel; kSrcBitmap only names that
// source for the host code.)
constexpr int kSrcBf16 = 0, kSrcFp32 = 1, kSrcBitmap = 2;

// Waves per SIMD are demanded where a few registers more would cost one; of the present kernels only lists of one-byte elements in
// tiles of 16384 would have one fewer without.  7 waves / 8, us: five 32B-shaped layers in place at 0.3 % 1247 / 1206, rotated
// 1089 / 1040, four 8B-shaped 519 / 522, one of them 132 / 136.
constexpr int waves_per_simd(int v, bool multi, int src, int eb) {
    return (v >= 16 && src == kSrcBf16) ? 3 : (v == 8 && src == kSrcFp32) ? 4 : (v == 4 && eb == 1 && multi) ? 8 : 1;
}

// 16 bytes moved up / down by `bytes` (0 .. 15), zeros coming in
__device__ __forceinline__ u32x4 shift_up(u32x4 v, uint32_t bytes) {
    unsigned long long lo = ((unsigned long long)v.y << 32) | v.x, hi = ((unsigned long long)v.w << 32) | v.z;
    const uint32_t n = (bytes & 7u) * 8u;
    if (bytes >= 8u) { hi = lo; lo = 0; }
    hi = (hi << n) | (n ? lo >> (64u - n) : 0ull);
    lo <<= n;
    u32x4 r;
    r.x = (uint32_t)lo; r.y = (uint32_t)(lo >> 32); r.z = (uint32_t)hi; r.w = (uint32_t)(hi >> 32);
    return r;
}
__device__ __forceinline__ u32x4 shift_down(u32x4 v, uint32_t bytes) {
    unsigned long long lo = ((unsigned long long)v.y << 32) | v.x, hi = ((unsigned long long)v.w << 32) | v.z;
    const uint32_t n = (bytes & 7u) * 8u;
    if (bytes >= 8u) { lo = hi; hi = 0; }
    lo = (lo >> n) | (n ? hi << (64u - n) : 0ull);
    hi >>= n;
    u32x4 r;
    r.x = (uint32_t)lo; r.y = (uint32_t)(lo >> 32); r.z = (uint32_t)hi; r.w = (uint32_t)(hi >> 32);
    return r;
}

template <int V, bool MULTI, int RG, int SRC, int EB, bool WHOLE>
__device__ __forceinline__ void extract_tile(const ExtractArgs &a) {
    // A snapshot that is not written is read exactly once, like the new weights: both streams then carry the
    // non-temporal hint (measured 4 % faster).  With element-wise refresh the hint on either stream measures slower,
    // on the snapshot by 5 ms: 2-byte refresh stores must find their line still cached, hinted or not.
    static_assert(RG == -1 || RG == 0 || RG == 8, "refresh: none, element-wise or whole lines");
    constexpr bool NT = (RG < 0);
    constexpr bool LINES = (RG == 8);
    constexpr bool CAST = (SRC == kSrcFp32);
    static_assert(SRC == kSrcBf16 || SRC == kSrcFp32, "the bitmap source has its own kernel");
    static_assert(V % 2 == 0, "counts are scanned in packed pairs");
    static_assert(EB == 2 || SRC == kSrcBf16, "the cast flavour exists for 16-bit elements only");
    typedef Elem<EB> EL;
    typedef typename EL::type T;
    constexpr uint32_t VE = 16u / EB;                    // elements per 16-byte vector
    constexpr uint32_t ROW = 64u * VE;                   // elements covered by one load instruction of a wave
    constexpr uint32_t TILE = (uint32_t)V * kThreads * VE;
    static_assert(TILE <= 65536u, "tile-local positions are staged in 16 bits");
    __shared__ uint32_t s_ticket;
    __shared__ uint32_t s_wave_total[kWaves];
    __shared__ uint32_t s_excl;
    __shared__ uint32_t s_stage[kStage];
    __shared__ u32x4 s_tail;               // the tile's last, incomplete vector (see below) and its change mask
    __shared__ uint32_t s_tail_mask;

    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = uniform((uint32_t)tid >> 6), wbase = wave * (V * ROW);   // first grid position of the wave

    // ---- which bucket this workgroup serves, then claim that bucket's next tile
    uint32_t bucket, first_tile, bucket_tiles;
    if (MULTI) {
        const auto *wi = as_table(a.wg_info + blockIdx.x);
        bucket = wi->bucket; first_tile = wi->first_tile; bucket_tiles = wi->ntiles;
    } else {
        // groups of `group` buckets; inside a group consecutive workgroups rotate over its buckets.
        // Only the very last bucket may have fewer tiles: in its group the first last_tiles rounds
        // rotate over all buckets, the remaining rounds over all but the last.
        const uint32_t per_group = a.group * a.tiles_per_bucket;
        const uint32_t g = blockIdx.x / per_group;
        const uint32_t j = blockIdx.x - g * per_group;
        const uint32_t g0 = g * a.group;
        const uint32_t gb = (a.nb - g0 < a.group) ? (a.nb - g0) : a.group;      // buckets in this group
        const bool has_short = (g0 + gb == a.nb) && (a.last_tiles < a.tiles_per_bucket);
        uint32_t slot;
        if (!has_short || j < a.last_tiles * gb) slot = j % gb;
        else slot = (j - a.last_tiles * gb) % (gb - 1);
        bucket = g0 + slot;
        first_tile = bucket * a.tiles_per_bucket;
        bucket_tiles = (bucket == a.nb - 1) ? a.last_tiles : a.tiles_per_bucket;
    }
    // a bucket of one tile needs neither ticket nor status word
    uint32_t k = 0, epoch = 0;
    const bool chained = bucket_tiles > 1; // uniform
    if (chained) {
        epoch = launch_epoch(a);
        if (tid == 0) s_ticket = claim_tile(a, bucket, bucket_tiles);
        __syncthreads();
        k = uniform(s_ticket);
        if (k >= bucket_tiles) {           // only where calls that share the counters overlapped: the tile is lost
            if (tid == 0) atomicOr(a.flags, a.timeout);
            return;
        }
    }
    const uint32_t tile = first_tile + k;
    const bool last = (k == bucket_tiles - 1);
    const uint32_t found = (chained && k == 0) ? left_behind(a, tile) : 0u;

    // ---- where this tile lives
    constexpr uint32_t NB = CAST ? 4u : (uint32_t)EB;                   // bytes per new weight
    uint32_t len, idx_base;
    gptr<T> po; gptr<const uint8_t> pn;
    if (MULTI) {
        const auto *d = table<!WHOLE>(a.tiles + tile);
        const uint32_t tensor = d->tensor, off = d->tensor_off;
        len = d->len;
        idx_base = d->bucket_off;                       // index = position inside the bucket
        const auto *t = table<!WHOLE>(a.ptrs + tensor);
        po = (gptr<T>)t->old_w + off;
        pn = (gptr<const uint8_t>)as_global(t->new_w) + (uint64_t)off * NB;
    } else {
        const uint64_t b0 = (uint64_t)bucket * a.be;
        const uint32_t blen = (uint32_t)((a.n - b0 < a.be) ? (a.n - b0) : a.be), off = k * TILE;
        len = (blen - off < TILE) ? (blen - off) : TILE;
        po = (gptr<T>)a.old_w + b0 + off;
        pn = (gptr<const uint8_t>)as_global(a.new_w) + (b0 + off) * NB;
        idx_base = (uint32_t)(b0 + off);                // index = tensor-flat position
    }

    // ---- stream the tile in 16-byte vectors on a grid that starts at the 16-byte boundary at or before its first
    // snapshot element, h elements earlier.  Wave w owns grid positions [w*V*ROW, (w+1)*V*ROW); inside it vector j of
    // lane l holds positions (j*64 + l)*VE .. +VE, so ascending order is (wave, j, lane, element).  Vectors that lie
    // wholly in the tile are one load each whatever the alignment of the new weights.  What is left over is at most one
    // incomplete vector in front (thread 0's first) and one behind the last whole vector (thread kThreads-1 takes it, as
    // a vector of its own that ranks after all others).  Those two are read as the tile's first and last 16 bytes, at any
    // address, and shifted to their place; a tile shorter than a vector is read element by element.
    // All loads of a tile are in flight together: lanes that have no vector read the tile's first 16 bytes as well, and a tile
    // shorter than a vector reads the flag word.  Measured with what follows below, us, extract only, element by element / so:
    // 300 odd-sized tensors end to end (108 M elements, 1 % changed) 119 / 106, with the snapshot rotated and the new weights six
    // bytes off 98 / 80.  Whole tiles have a run of loads without a branch; in the others a wave leaves out fours of vectors that
    // it has none of, and does not pace what is left.  One run for both was slower wherever tiles are short, us: those 300
    // tensors in buckets of 9000 elements at 5 % in place 222 / 170, of 3000 at 1 % 441 / 295, cast in buckets of 9000 283 / 247,
    // one tensor of 1000 elements 3.5 / 3.3; and it took a spill in tiles of 16384 with masters and one-byte elements.
    u32x4 xo[V], xn[V], f1[CAST ? V : 1], to, tn, tn1;                   // f1, tn1: second halves of master vectors; to, tn: the tail
    const uint32_t h = (uint32_t)((uintptr_t)po & 15u) / EB;
    const uint32_t glen = len + h;                                      // grid positions h .. glen-1 exist
    const uint32_t nbody = (glen < TILE ? glen : TILE) / VE * VE;       // positions below it form whole vectors (but for h)
    uint32_t lv = (uint32_t)lane * VE;                                  // this lane's first position, from its wave's first
    auto fresh = [&]() { asm volatile("" : "+v"(lv)); };                // what follows derives its positions anew instead of keeping them in registers
    const uint32_t nw = nbody > wbase ? nbody - wbase : 0u;             // the wave's positions below it form whole vectors
    // bases of the grid: only positions h .. glen-1 are ever accessed
    const gptr<T> og = po - h;
    const gptr<const uint32_t> fg = (gptr<const uint32_t>)pn - h;     // with CAST: the master weights
    const gptr<const T> ng = (gptr<const T>)pn - h;
    const bool in_head = h != 0 && tid == 0;                            // this thread's first vector is the incomplete one in front
    const bool has_tail = glen > nbody;                                 // uniform
    const bool short_tile = len < VE;                                   // uniform
    const u32x4 none = {0u, 0u, 0u, 0u};
    constexpr bool H = NT || LINES;
    uint32_t m[V], ex[V], counted = 0;
    auto pace = [&](auto on) {
        constexpr int C = !decltype(on)::value || RG < 0 ? 0 : CAST ? kLoadPace / 2 : kLoadPace;
        if constexpr (C > 0) {
            __builtin_amdgcn_sched_barrier(0); __builtin_amdgcn_s_sleep(C); __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto refresh_incomplete = [&](uint32_t at, uint32_t mm, u32x4 x) {      // element by element
        for (; mm; mm &= mm - 1u) {
            const uint32_t e = (uint32_t)__builtin_ctz(mm);
            og[at + e] = (T)EL::pattern(x, e);
        }
    };
    if constexpr (WHOLE) {
        // Lists nearly all of whose tiles are whole and lie on the 16-byte boundaries: addresses per lane with immediate offsets,
        // tables by vector loads, and nothing in the way of the other tiles, which are read as simply as can be: even the
        // branch around the other form's code costs such a list up to 1 %.  Where the host takes which is said there.
        static_assert(!CAST && EB == 2, "16-bit weights on both sides");
        const uint32_t g0 = ((uint32_t)tid >> 6) * (V * ROW) + (uint32_t)lane * VE;
        if (h == 0 && glen == TILE) {
#pragma unroll
            for (int j = 0; j < V; ++j) { xn[j] = load16_any<H>(ng + g0 + j * ROW); pace(std::true_type{}); }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < V; ++j) { xo[j] = load16<H>(og + g0 + j * ROW); pace(std::true_type{}); }
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const uint32_t g = g0 + j * ROW;
                const bool there = g < nbody && (j > 0 || !in_head);
                xo[j] = there ? load16<H>(og + g) : none;
                xn[j] = there ? load16_any<H>(ng + g) : none;
            }
            const bool front = in_head && nbody != 0;
            if (front || (has_tail && tid == kThreads - 1)) {
                const uint32_t at = front ? 0u : nbody;
                const uint32_t lo = (h > at) ? h - at : 0u, hi = front ? VE : glen - nbody;
                const u32x4 vo = EL::load_window(og + at, lo, hi), vn = EL::load_window(ng + at, lo, hi);
                if (front) { xo[0] = vo; xn[0] = vn; }
                const uint32_t md = EL::diff_mask(vo, vn);
                if (!front) { s_tail = vn; s_tail_mask = md; }
                if (LINES) refresh_incomplete(at, md, vn);
            }
        }
        if (chained && last && tid == 0) counted = count_claimed(a);           // returns with the loads
#pragma unroll
        for (int j = 0; j < V; ++j) m[j] = EL::diff_mask(xo[j], xn[j]);
    } else {
        auto stream_tile = [&](auto whole) {
            constexpr bool W = decltype(whole)::value;           // every vector exists, but for thread 0's first
            const gptr<const uint8_t> ob = scalar_base(!W && short_tile ? (gptr<const uint8_t>)as_global(a.flags) : (gptr<const uint8_t>)og);
            const gptr<const uint8_t> nb = scalar_base(!W && short_tile ? (gptr<const uint8_t>)as_global(a.flags)
                                                       : CAST ? (gptr<const uint8_t>)fg : (gptr<const uint8_t>)ng);
            const uint32_t spare = !W && short_tile ? 0u : h;
            auto has_vector = [&](int j) -> bool { return (W || lv + j * ROW < nw) && !(j == 0 && in_head); };
            auto position = [&](int j) -> uint32_t { return (W && j) || has_vector(j) ? wbase + lv + j * ROW : spare; };
            constexpr int G = V < 4 ? V : 4;                     // an incomplete tile loads or leaves out so many vectors together
            __builtin_amdgcn_sched_barrier(0);
            uint32_t t_pos = has_tail && !short_tile ? glen - VE : spare;
            asm volatile("" : "+v"(t_pos));       // uniform: the compiler would wait for the loads to move them to scalar registers
            tn = load16_any<false>(nb + t_pos * NB);
            if (CAST) tn1 = load16_any<false>(nb + (t_pos * NB + 16u));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < V; i += G) {
                if (W || i * ROW < nw) {
#pragma unroll
                    for (int j = i; j < i + G; ++j) {
                        xn[j] = load16_any<H && !CAST>(nb + position(j) * NB); pace(whole);
                        if (CAST) { f1[j] = load16_any<false>(nb + (position(j) * NB + 16u)); pace(whole); }
                    }
                } else {
#pragma unroll
                    for (int j = i; j < i + G; ++j) { xn[j] = none; if (CAST) f1[j] = none; }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            fresh();
            to = load16_any<false>(ob + t_pos * (uint32_t)EB);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < V; i += G) {
                if (W || i * ROW < nw) {
#pragma unroll
                    for (int j = i; j < i + G; ++j) { xo[j] = load16_any<H>(ob + position(j) * (uint32_t)EB); pace(whole); }
                } else {
#pragma unroll
                    for (int j = i; j < i + G; ++j) xo[j] = none;
                }
            }
            if (chained && last && tid == 0) counted = count_claimed(a);           // returns with the loads
            fresh();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if (CAST) xn[j] = round8_bf16(xn[j], f1[j]);
                m[j] = EL::diff_mask(xo[j], xn[j]);
                if (!W && !has_vector(j)) m[j] = 0;
                if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (glen >= TILE) stream_tile(std::true_type{});
        else stream_tile(std::false_type{});

        if (in_head) {
            // the front: elements 0 .. VE-h-1 of the tile, to positions h .. VE-1
            u32x4 vo, vn;
            if (short_tile) {
                const uint32_t hi = glen < VE ? 0u : VE;                    // (a tile within one vector is all tail)
                vo = EL::load_window(og, h, hi);
                if constexpr (CAST) vn = load8_window_cast(fg, h, hi);
                else vn = EL::load_window(ng, h, hi);
            } else {
                vo = shift_up(xo[0], h * EB);
                vn = shift_up(xn[0], h * EB);
            }
            xn[0] = vn;
            m[0] = EL::diff_mask(vo, vn);
            if (LINES) refresh_incomplete(0, m[0], vn);
        }
        if (has_tail && tid == kThreads - 1) {
            uint32_t md;
            u32x4 vn;
            if (short_tile) {
                const uint32_t lo = (h > nbody) ? h - nbody : 0u, hi = glen - nbody;
                const u32x4 vo = EL::load_window(og + nbody, lo, hi);
                if constexpr (CAST) vn = load8_window_cast(fg + nbody, lo, hi);
                else vn = EL::load_window(ng + nbody, lo, hi);
                md = EL::diff_mask(vo, vn);
            } else {
                const uint32_t down = (VE - (glen - nbody)) * EB;
                if (CAST) tn = round8_bf16(tn, tn1);
                vn = shift_down(tn, down);
                md = EL::diff_mask(shift_down(to, down), vn);
            }
            s_tail = vn;
            s_tail_mask = md;
            if (LINES) refresh_incomplete(nbody, md, vn);
        }
    }

    // ---- wave scan (two vectors per register), then the rank of this lane's first changed element of each vector
    uint32_t wave_total = 0;
#pragma unroll
    for (int q = 0; q < V / 2; ++q) {
        const uint32_t both = __popc(m[2 * q]) | (__popc(m[2 * q + 1]) << 16);
        uint32_t inc = wave_inclusive_scan(both);
        asm("" : "+v"(inc));                 // inc - both stays a difference: as a sum of the scan's steps it would keep six registers
        const uint32_t tot = lane63(inc), exc = inc - both;
        ex[2 * q] = wave_total + (exc & 0xFFFFu);
        wave_total += tot & 0xFFFFu;
        ex[2 * q + 1] = wave_total + (exc >> 16);
        wave_total += tot >> 16;
    }
    if (LINES) refresh_lines<V, T>(og, wbase + lv, nbody, in_head, m, xn, lane);
    fresh();
    if (lane == 0) s_wave_total[wave] = wave_total;
    __syncthreads();
    uint32_t wave_base = 0, tile_total = 0;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)kWaves; ++w) {
        const uint32_t t = uniform(s_wave_total[w]);
        wave_base += (w < wave) ? t : 0u;
        tile_total += t;
    }
    const uint32_t tail_rank = tile_total;                // the tail's changed elements rank last
    const uint32_t tail_mask = has_tail ? uniform(s_tail_mask) : 0u;
    tile_total += (uint32_t)__popc(tail_mask);
#pragma unroll
    for (int j = 0; j < V; ++j) ex[j] += wave_base;       // from here on: rank inside the tile

    // ---- the chain with the earlier tiles of the bucket: this tile's count is published now, and looked back from later
    if (tid == 0) {
        if (chained) publish(a, epoch, tile, found, tile == first_tile, last, tile_total);
        else if (a.chained) wipe_alone(a, tile);
    }
    // wave 0: changed elements of the bucket in front of the tile
    auto settle = [&]() -> uint32_t {
        uint32_t excl = 0;
        if (tile != first_tile) {
            excl = look_back(a, epoch, tile, first_tile, lane);
            if (lane == 0 && !last) status_store(a.status + tile, status_word(epoch, kStPrefix, excl + tile_total));
        }
        if (last) {
            const uint32_t c = excl + tile_total;
            if (lane == 0) {
                a.counts[bucket] = c;
                if ((uint64_t)c > a.cap) atomicOr(a.flags, kFlagOverflow);
            }
            if (chained) raise_epoch(a, epoch, counted, lane);
        }
        return excl;
    };

    int32_t *const Ib = a.I + (uint64_t)bucket * a.cap;
    T *const Vb = reinterpret_cast<T *>(a.V) + (uint64_t)bucket * a.cap;
    auto write_staged = [&](uint32_t from, uint32_t step, uint64_t rank0, uint32_t n) {
        for (uint32_t q = from; q < n; q += step) {
            const uint32_t ent = s_stage[q];
            const uint32_t local = ent >> 16;
            const T val = (T)(ent & 0xFFFFu);
            const uint64_t r = rank0 + q;
            if (local < len) {                      // always true for a correct scan; keeps stores in bounds
                if (r < a.cap) { Ib[r] = (int32_t)(idx_base + local); Vb[r] = val; }
                if (RG == 0) po[local] = val;           // snapshot refresh: W_prev <- W at changed positions
            }
        }
    };
    auto stage_round = [&](uint32_t r0) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            uint32_t mm = m[j];
            // the ranks of this vector's changed elements are ex[j] .. ex[j] + popc - 1: nothing to do in a round
            // that lies wholly before or after them (this keeps dense tiles linear in the number of rounds)
            if (mm && ex[j] < r0 + kStage && ex[j] + __popc(mm) > r0) {
                uint32_t rank = ex[j] - r0;                  // wraps for elements of earlier rounds: skipped below
                const uint32_t local = wbase + j * ROW - h + lv;
                while (mm) {
                    const uint32_t e = (uint32_t)__builtin_ctz(mm);
                    mm &= mm - 1u;
                    if (rank < kStage) s_stage[rank] = ((local + e) << 16) | EL::pattern(xn[j], e);
                    ++rank;
                }
            }
        }
        if (has_tail && tid == kThreads - 1) {
            uint32_t rank = tail_rank - r0;
            for (uint32_t mm = tail_mask; mm; mm &= mm - 1u, ++rank) {
                const uint32_t e = (uint32_t)__builtin_ctz(mm);
                if (rank < kStage) s_stage[rank] = ((nbody - h + e) << 16) | EL::pattern(s_tail, e);
            }
        }
    };

    if (tile_total <= kStage) {
        // One round of pairs, the usual case.  A tile's place in its bucket is known when all tiles before it have been
        // counted, and where few buckets share the card hundreds of tiles wait for the slowest of them.  So the pairs are
        // staged first, which gives the others time to publish and saves most polls of the status words; then three of
        // the four waves end and give their registers back to workgroups that can load; wave 0 alone waits and writes out.
        // Looking back at once / after staging / and with three waves gone, us: one 8B-shaped layer at 0.6 % refreshed in
        // place 184 / 170 / 166 and rotated 159 / 147 / 143, 311 M elements in one bucket at 1 % 315 / 292 / 283 and
        // 263 / 237 / 232, the same in 64 buckets 283 / 283 / 282.  (A workgroup that goes on to further tiles while the
        // last ones wait in LDS gains as much on one bucket, but loses 3 to 7 % on many and a third on dense data.)
        // All four waves write where nothing is waited for, in the only tile of its bucket, and where the pairs are many: one
        // wave alone takes 2048 of them out in 32 turns.  One wave / four, us: one tensor of 16 K one-byte elements at 5 % in
        // place 6.4 / 5.3, 1000 elements at 40 % 4.9 / 4.4, nine buckets of 1820 at 40 % rotated 5.3 / 4.7; more than 1024 pairs
        // in a tile of the largest size: 8B-shaped layers rotated at 5 %, one 157 / 155, four 541 / 525; 30B-A3B-shaped, one of
        // them -2 %, six -1 %.  (From 256 pairs on a tile one 8B-shaped layer at 1 % loses 1 %.)
        stage_round(0);
        lds_barrier();
        if (!chained) {
            if (wave == 0) settle();
            write_staged((uint32_t)tid, kThreads, 0, tile_total);
            return;
        }
        if (V >= 16 && tile_total > kStage / 2) {
            if (wave == 0) {
                const uint32_t e = settle();
                if (lane == 0) s_excl = e;
            }
            lds_barrier();
            write_staged((uint32_t)tid, kThreads, uniform(s_excl), tile_total);
            return;
        }
        if (wave != 0) return;
        const uint32_t excl = settle();
        write_staged((uint32_t)lane, 64, excl, tile_total);
        return;
    }
    if (wave == 0) {
        const uint32_t e = settle();
        if (lane == 0) s_excl = e;
    }
    __syncthreads();
    const uint32_t excl = uniform(s_excl);
    if (V >= 16) {
        // The largest tiles leave room for three workgroups per CU at most, and on dense data (several rounds of
        // staging) those spend most of their time writing out, with no loads in flight.  There every thread writes its
        // own pairs at their ranks instead: the lanes of a wave hold consecutive rank ranges, so these stores are
        // close together, and no round needs a barrier (measured at 25 % / 100 % density: 12.7 / 34.8 ms against
        // 22.3 / 39.9 ms staged; smaller tiles do better staged).
        auto write_out = [&](uint32_t mm, uint32_t r, uint32_t g, u32x4 x) {
            // r is below 2^32: a bucket holds fewer than 2^31 elements
            while (mm) {
                const uint32_t e = (uint32_t)__builtin_ctz(mm);
                mm &= mm - 1u;
                const T val = (T)EL::pattern(x, e);
                const uint32_t local = g + e - h;
                if (local < len) {                  // masks are zero outside the tile; keeps stores in bounds regardless
                    if ((uint64_t)r < a.cap) { Ib[r] = (int32_t)(idx_base + local); Vb[r] = val; }
                    if (RG == 0) po[local] = val;
                }
                ++r;
                // 8 clocks between the pairs of the kernel that also rewrites lines: its stores then leave more evenly, as its
                // loads do.  Refreshed by lines, without / with, us: two 32B-shaped layers at 10 % 1261 / 1272, 30 % 1746 /
                // 1670, 50 % 2338 / 2261, 100 % 4278 / 4388; three 30B-A3B-shaped at 30 % 3005 / 2944.  (16 and 32 clocks
                // gain more at 50 % and lose 1 to 2 % at 20 %.)
                if (LINES) asm volatile("s_nop 7");
            }
        };
#pragma unroll
        for (int j = 0; j < V; ++j) write_out(m[j], excl + ex[j], wbase + j * ROW + lv, xn[j]);
        if (has_tail && tid == kThreads - 1) write_out(tail_mask, excl + tail_rank, nbody, s_tail);
        return;
    }
    // The barriers of this loop order LDS accesses only (lds_barrier): a full __syncthreads would also wait for the round's
    // global stores to complete, which on dense tiles (many rounds) costs more than the stores themselves.
    for (uint32_t r0 = 0; r0 < tile_total; r0 += kStage) {
        stage_round(r0);
        lds_barrier();
        write_staged((uint32_t)tid, kThreads, (uint64_t)excl + r0, (tile_total - r0 < kStage) ? (tile_total - r0) : kStage);
        lds_barrier();
    }
}

template <int V, bool MULTI, int RG, int SRC = kSrcBf16, int EB = 2>
__global__ __launch_bounds__(kThreads, waves_per_simd(V, MULTI, SRC, EB)) void extract_kernel(const ExtractArgs a) {
    extract_tile<V, MULTI, RG, SRC, EB, false>(a);
}

// for lists nearly all of whose tiles are whole and aligned
template <int RG>
__global__ __launch_bounds__(kThreads, waves_per_simd(16, true, kSrcBf16, 2)) void extract_whole_kernel(const ExtractArgs a) {
    extract_tile<16, true, RG, kSrcBf16, 2, true>(a);
}

// ---------------------------------------------------------------------------------------------
// extract_marked_kernel: Alg. 2's V = W[I] over the cumulative index set of Alg. 1, held as a bitmap over packed
// positions (mark_kernel builds it).  The bitmap already says where the changes are, so the weights are not
// streamed: the workgroup reads its tile's slice of the bitmap (one bit per element), ranks the set bits like
// extract_kernel ranks changed elements (wave scan, LDS combine, the same per-bucket ticket and look-back chain),
// stages their tile-local positions in LDS in rank order, and only then fetches the values, one 2-byte gather
// per pair, balanced over the 256 threads and written out coalesced next to the indices.  Memory traffic is the
// bitmap plus the lines that hold a marked element instead of the whole weight set.
// E = elements per thread (tile of the plan / 256); thread t owns the tile-local positions [t*E, (t+1)*E).  NT: the gathers
// carry the non-temporal hint.
// ---------------------------------------------------------------------------------------------

// the nbits (1..32) bitmap bits of packed positions g .. g+nbits-1, bit k of the result for position g + k
__device__ __forceinline__ uint32_t bitmap_bits32(const uint32_t *bitmap, uint64_t words, uint64_t g, uint32_t nbits) {
    const uint64_t w = g >> 5;
    const uint32_t sh = (uint32_t)(g & 31u);
    const uint32_t lo = bitmap[w];
    const uint32_t hi = (sh != 0u && sh + nbits > 32u && w + 1 < words) ? bitmap[w + 1] : 0u;
    const uint32_t bits = (uint32_t)((((unsigned long long)hi << 32) | lo) >> sh);
    return nbits >= 32u ? bits : (bits & ((1u << nbits) - 1u));
}

template <int E, bool NT>
__global__ __launch_bounds__(kThreads) void extract_marked_kernel(const ExtractArgs a) {
    static_assert(E == 16 || E == 32 || E == 64 || E == 128, "tile of 4096 .. 32768 elements");
    constexpr int NW = (E + 31) / 32;                    // mask words per thread
    constexpr uint32_t CH = (E < 32) ? (uint32_t)E : 32u; // elements per mask word
    constexpr int kGather = (int)(kStage / kThreads);    // gathers in flight per thread
    static_assert(E * kThreads <= 65536, "positions and values share a word");
    __shared__ uint32_t s_ticket;
    __shared__ uint32_t s_wave_total[kWaves];
    __shared__ uint32_t s_excl;
    __shared__ uint32_t s_stage[kStage];                 // tile-local positions in rank order, then position << 16 | value

    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = uniform((uint32_t)tid >> 6);

    // ---- bucket, ticket, tile: as in extract_kernel (tensor lists only)
    const auto *wi = as_table(a.wg_info + blockIdx.x);
    const uint32_t bucket = wi->bucket, first_tile = wi->first_tile, bucket_tiles = wi->ntiles;
    uint32_t k = 0, epoch = 0;
    const bool chained = bucket_tiles > 1;
    if (chained) {
        epoch = launch_epoch(a);
        if (tid == 0) s_ticket = claim_tile(a, bucket, bucket_tiles);
        __syncthreads();
        k = uniform(s_ticket);
        if (k >= bucket_tiles) {           // as in extract_kernel
            if (tid == 0) atomicOr(a.flags, a.timeout);
            return;
        }
    }
    const uint32_t tile = first_tile + k;
    const bool last = (k == bucket_tiles - 1);
    const uint32_t found = (chained && k == 0) ? left_behind(a, tile) : 0u;
    const auto *d = as_table(a.tiles + tile);
    const uint32_t tensor = d->tensor, tensor_off = d->tensor_off, len = d->len, idx_base = d->bucket_off;
    const gptr<const uint16_t> pn = (gptr<const uint16_t>)as_global(as_table(a.ptrs + tensor)->new_w) + tensor_off;
    const uint64_t g0 = *as_table(a.tensor_base + tensor) + tensor_off;      // packed position of the tile's first element

    // ---- this thread's slice of the bitmap and its count: one 16-byte load and the word behind it where the slice is whole
    const uint32_t e0 = (uint32_t)tid * E;
    uint32_t m[NW];
    uint32_t mine = 0;
    const uint64_t w0 = (g0 + e0) >> 5;
    const uint32_t sh = (uint32_t)(g0 & 31u);            // e0 is a multiple of 32 there
    if (NW == 4 && e0 + E <= len && w0 + 4 < a.bitmap_words) {
        const u32x4 q = load16_any<false>((gptr<const uint32_t>)a.bitmap + w0);
        const uint32_t next = a.bitmap[w0 + 4];
        const uint32_t x[5] = {q.x, q.y, q.z, q.w, next};
#pragma unroll
        for (int c = 0; c < NW; ++c) m[c] = (uint32_t)((((unsigned long long)x[c + 1] << 32) | x[c]) >> sh);
    } else {
#pragma unroll
        for (int c = 0; c < NW; ++c) {
            const uint32_t e = e0 + c * 32u;
            const uint32_t left = (e < len) ? (len - e) : 0u;
            const uint32_t nbits = left < CH ? left : CH;
            m[c] = nbits ? bitmap_bits32(a.bitmap, a.bitmap_words, g0 + e, nbits) : 0u;
        }
    }
#pragma unroll
    for (int c = 0; c < NW; ++c) mine += __popc(m[c]);
    uint32_t counted = 0;
    if (chained && last && tid == 0) counted = count_claimed(a);     // returns behind the bitmap
    const uint32_t inc = wave_inclusive_scan(mine);                  // at most 64 * 128 per wave
    const uint32_t wave_total = lane63(inc);
    if (lane == 0) s_wave_total[wave] = wave_total;
    __syncthreads();
    uint32_t wave_base = 0, tile_total = 0;
#pragma unroll
    for (uint32_t w = 0; w < (uint32_t)kWaves; ++w) {
        const uint32_t t = uniform(s_wave_total[w]);
        wave_base += (w < wave) ? t : 0u;
        tile_total += t;
    }
    const uint32_t first = wave_base + (inc - mine);                 // rank of this thread's first pair

    // ---- chain with the earlier tiles of the bucket, as in extract_kernel: published now, looked back from later
    if (tid == 0) {
        if (chained) publish(a, epoch, tile, found, tile == first_tile, last, tile_total);
        else if (a.chained) wipe_alone(a, tile);
    }
    auto settle = [&]() -> uint32_t {
        uint32_t excl = 0;
        if (tile != first_tile) {
            excl = look_back(a, epoch, tile, first_tile, lane);
            if (lane == 0 && !last) status_store(a.status + tile, status_word(epoch, kStPrefix, excl + tile_total));
        }
        if (last) {
            const uint32_t c = excl + tile_total;
            if (lane == 0) {
                a.counts[bucket] = c;
                if ((uint64_t)c > a.cap) atomicOr(a.flags, kFlagOverflow);
            }
            if (chained) raise_epoch(a, epoch, counted, lane);
        }
        return excl;
    };

    int32_t *const Ib = a.I + (uint64_t)bucket * a.cap;
    uint16_t *const Vb = a.V + (uint64_t)bucket * a.cap;
    // positions of the pairs r0 .. r0 + kStage - 1 into LDS in rank order
    auto stage_round = [&](uint32_t r0) {
        uint32_t rank = first - r0;                                  // wraps for pairs of earlier rounds: skipped below
        const bool in_round = first < r0 + kStage && first + mine > r0;   // this thread has pairs of this round
#pragma unroll
        for (int c = 0; c < NW; ++c) {
            uint32_t mm = in_round ? m[c] : 0u;
            while (mm) {
                const uint32_t e = (uint32_t)__builtin_ctz(mm);
                mm &= mm - 1u;
                if (rank < kStage) s_stage[rank] = e0 + c * 32u + e;
                ++rank;
            }
        }
    };
    // their values, spread evenly over the threads and all in flight together, go back to LDS beside the positions
    auto gather_round = [&](uint32_t n) {
        if (n <= (uint32_t)kThreads) {                                  // one each (uniform)
            const uint32_t q = (uint32_t)tid;
            if (q < n) {
                const uint32_t local = s_stage[q];
                uint32_t val = 0;
                if (local < len) val = NT ? __builtin_nontemporal_load(pn + local) : pn[local];
                s_stage[q] = (local << 16) | val;
            }
            return;
        }
        uint32_t local[kGather], val[kGather];
#pragma unroll
        for (int u = 0; u < kGather; ++u) {
            const uint32_t q = (uint32_t)tid + u * kThreads;
            local[u] = 0;
            val[u] = 0;
            if (q < n) local[u] = s_stage[q];
            if (q < n && local[u] < len) val[u] = NT ? __builtin_nontemporal_load(pn + local[u]) : pn[local[u]];
        }
#pragma unroll
        for (int u = 0; u < kGather; ++u) {
            const uint32_t q = (uint32_t)tid + u * kThreads;
            if (q < n) s_stage[q] = (local[u] << 16) | val[u];
        }
    };
    auto write_staged = [&](uint32_t from, uint32_t step, uint64_t rank0, uint32_t n) {
        for (uint32_t q = from; q < n; q += step) {
            const uint32_t ent = s_stage[q], local = ent >> 16;
            const uint64_t r = rank0 + q;
            if (local < len && r < a.cap) { Ib[r] = (int32_t)(idx_base + local); Vb[r] = (uint16_t)(ent & 0xFFFFu); }
        }
    };

    if (tile_total <= kStage) {
        // The values do not wait for the tile's place in the bucket; when they are there, three of the four waves end, and
        // wave 0 looks back and writes out.  (Before, the gathers waited for the look-back: the chain of latencies from the
        // bitmap's address to the payload bounds this kernel, at eight workgroups per CU.)  Before / now, us: four
        // 30B-A3B-shaped layers at 1.2 % marked 752 / 653, four 32B-shaped at 0.07 % 297 / 197, eight 8B-shaped at 3 % 667 / 607,
        // one at 0.6 % 50 / 41, 300 odd-sized tensors at 2 % 43 / 33; with all four waves to the end 701 for the first.
        stage_round(0);
        lds_barrier();
        // A pair each at most and nothing to wait for: out they go.  With all of what follows for such tiles too the extract of 600
        // tensors in buckets of 3000 elements took 141 us at 0.2 % marked and 197 at 2 %, where it had taken 129 and 179 before the
        // values went through LDS; so 131 and 187.
        if (!chained && tile_total <= (uint32_t)kThreads) {
            if ((uint32_t)tid < tile_total) {
                const uint32_t local = s_stage[tid];
                if (local < len && (uint32_t)tid < a.cap) {
                    const uint16_t val = NT ? __builtin_nontemporal_load(pn + local) : pn[local];
                    Ib[tid] = (int32_t)(idx_base + local);
                    Vb[tid] = val;
                }
            }
            if (wave == 0) settle();
            return;
        }
        gather_round(tile_total);
        lds_barrier();
        if (wave != 0) return;
        const uint32_t excl = settle();
        write_staged((uint32_t)lane, 64, excl, tile_total);
        return;
    }
    if (wave == 0) {
        const uint32_t e = settle();
        if (lane == 0) s_excl = e;
    }
    __syncthreads();
    const uint32_t excl = uniform(s_excl);
    for (uint32_t r0 = 0; r0 < tile_total; r0 += kStage) {
        const uint32_t n = (tile_total - r0 < kStage) ? (tile_total - r0) : kStage;
        stage_round(r0);
        lds_barrier();
        gather_round(n);
        write_staged((uint32_t)tid, kThreads, (uint64_t)excl + r0, n);       // the thread's own entries
        lds_barrier();
    }
}

// ---------------------------------------------------------------------------------------------
// mark_kernel: one optimizer step of Alg. 1's index accumulation, I_cum <- I_cum U { i : W[i] != W_prev[i] },
// kept as a bitmap over packed positions.  CAST = false compares two BF16 versions; CAST = true is the
// Trainer's own sequence without the clone: W <- round_BF16(master) and the elements whose pattern changed
// are marked.  One workgroup per tile of the plan, in tile order; no chain, no ticket: tiles are independent here.
// (Extract's bucket-interleaved order measured 3 % faster for two BF16 versions and 5 % slower with CAST.)
// ---------------------------------------------------------------------------------------------
// Tiles are read on extract_kernel's grid of 16-byte vectors, so that any alignment and length takes whole vectors but for
// the incomplete ones in front and behind, which are read (and with CAST written back) element by element.  300 odd-sized
// tensors end to end, the buffers two bytes off (108 M elements, 1 % changed, two steps marked and extracted): 605 us when
// every vector of such a tile was read element by element, 208 us now.
// The bits are gathered in LDS first, so that the bitmap sees one coalesced atomic per 256 bytes of it and wave instead of one
// per vector that holds a change: two steps of 1.2 G elements marked and extracted, 0.6 % changed 2.06 -> 2.01 ms, 5 %
// 3.58 -> 2.36 ms, 0.1 % 1.82 ms as before.
template <int V, bool CAST>
__global__ __launch_bounds__(kThreads) void mark_kernel(const ExtractArgs a) {
    constexpr uint32_t TILE = (uint32_t)V * kUnit;
    constexpr uint32_t kWords = TILE / 32 + 4;           // 32 + 31 + TILE + 7 bits and the word that a last vector may spill into
    __shared__ uint32_t s_bits[kWords];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x >= a.ntiles) return;
    const TileDesc d = a.tiles[blockIdx.x];
    const PtrPair p = a.ptrs[d.tensor];
    const gptr<uint16_t> po = as_global(p.old_w) + d.tensor_off;
    const uint32_t len = d.len;
    const uint32_t h = (uint32_t)((uintptr_t)po & 15u) / 2;
    const uint32_t glen = len + h;                                      // grid positions h .. glen-1 exist
    const uint32_t nbody = (glen < TILE ? glen : TILE) / 8 * 8;         // positions below it form whole vectors (but for h)
    const uint32_t g0 = (uint32_t)wave * (V * 512u) + (uint32_t)lane * 8u;
    const gptr<uint16_t> og = po - h;
    const gptr<const uint32_t> fg = (gptr<const uint32_t>)p.new_w + d.tensor_off - h;
    const gptr<const uint16_t> ng = (gptr<const uint16_t>)p.new_w + d.tensor_off - h;
    // word 0 of s_bits is the one before the word of the tile's first element: grid positions below h are in front of it
    const uint64_t pos = a.tensor_base[d.tensor] + d.tensor_off;        // packed position of the tile's first element
    const uint32_t bit0 = 32u + (uint32_t)(pos & 31u) - h;              // bit of grid position 0 in s_bits
    for (uint32_t i = tid; i < kWords; i += kThreads) s_bits[i] = 0;
    __syncthreads();
    const bool in_head = h != 0 && tid == 0;
    u32x4 xo[V], xn[V];
    // two versions that are only compared are read once each: non-temporal (2 % faster); with CAST the parameters are
    // rewritten below by whole lines, hinted like extract's snapshot, and the master weights stay on ordinary loads
    auto load = [&](int j, uint32_t g) {
        xo[j] = load16<true>(og + g);
        if (CAST) xn[j] = round8_bf16(load16_any<false>(fg + g), load16_any<false>(fg + g + 4));
        else xn[j] = load16_any<true>(ng + g);
    };
    if (glen >= TILE) {                                                 // uniform over the workgroup
        // the thread of the incomplete vector reads its neighbour's instead (and its own below)
#pragma unroll
        for (int j = 0; j < V; ++j) load(j, (j == 0 && in_head) ? 8u : g0 + j * 512);
    } else {
        const u32x4 none = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const uint32_t g = g0 + j * 512;
            xo[j] = none; xn[j] = none;
            if (g < nbody && (j > 0 || !in_head)) load(j, g);
        }
    }
    auto mark = [&](uint32_t g, uint32_t m) {                           // bit k of m: grid position g + k changed
        const uint32_t at = bit0 + g, sh = at & 31u;
        atomicOr(&s_bits[at >> 5], m << sh);
        if (sh > 24u) atomicOr(&s_bits[(at >> 5) + 1], m >> (32u - sh));
    };
    const bool has_tail = glen > nbody;                                 // uniform
    if (h != 0 || has_tail) {
        const bool front = in_head && nbody != 0;
        if (front || (has_tail && tid == kThreads - 1)) {
            const uint32_t at = front ? 0u : nbody;
            const uint32_t lo = (h > at) ? h - at : 0u, hi = front ? 8u : glen - nbody;
            const u32x4 vo = load8_window(og + at, lo, hi);
            const u32x4 vn = CAST ? load8_window_cast(fg + at, lo, hi) : load8_window(ng + at, lo, hi);
            const uint32_t md = diff_mask8(vo, vn);
            if (front) { xo[0] = vo; xn[0] = vn; }
            else if (md) mark(at, md);
            if (CAST) {
                for (uint32_t mm = md; mm; mm &= mm - 1u) {
                    const uint32_t e = (uint32_t)__builtin_ctz(mm);
                    og[at + e] = (uint16_t)pattern_at(vn, e);
                }
            }
        }
    }
    uint32_t m[V];
#pragma unroll
    for (int j = 0; j < V; ++j) m[j] = diff_mask8(xo[j], xn[j]);
    if (CAST) refresh_lines<V, uint16_t>(og, g0, nbody, in_head, m, xn, lane);   // write the cast back where it changed something
#pragma unroll
    for (int j = 0; j < V; ++j)
        if (m[j]) mark(g0 + j * 512, m[j]);
    __syncthreads();
    uint32_t *const w = a.bitmap + (pos >> 5);
    for (uint32_t i = tid; i + 1 < kWords; i += kThreads) {
        const uint32_t x = s_bits[i + 1];
        if (x) atomicOr(w + i, x);                                      // bits are set for elements that exist only
    }
}

// ---------------------------------------------------------------------------------------------
// apply: W[I] <- V.  One workgroup per (bucket, chunk of kApplyChunk pairs); each thread owns
// kApplyPer pairs, kThreads apart, so that the index and value loads of a wave are contiguous and
// all of a thread's loads are in flight before its first store.  For tensor lists the bucket's
// segment table (start inside the bucket -> byte address of that element) is cached in LDS.
// ---------------------------------------------------------------------------------------------
constexpr int kApplyPer = (int)(kApplyChunk / kThreads);
constexpr uint32_t kSegCache = 128;
constexpr uint32_t kWideGap = 32768u;      // differences of 2^15 and more do not fit the 16-bit index coding

struct ApplyShared {
    uint32_t off[kSegCache + 1];
    unsigned long long base[kSegCache];
    uint32_t wave_total[kWaves];
};

// Common front of the apply kernels: which (bucket, chunk) this workgroup owns and how many of the
// chunk's pairs are valid; 0 when there is nothing to do.  Consecutive workgroups take the same chunk number of
// consecutive buckets (groups of kApplyInterleave buckets), so that the scatter of the moment is spread over the
// whole weight set instead of a dozen buckets: 12 % faster on the 910-bucket benchmark set at 1 %, 9 % at 5 %,
// nothing lost on the 244-bucket sets, 0.16 ms lost on the skewed set.
constexpr uint32_t kApplyInterleave = 1024;

__device__ __forceinline__ uint32_t apply_chunk(const ApplyArgs &a, uint32_t per_bucket, uint32_t &b, uint64_t &start) {
    const uint32_t per_group = kApplyInterleave * per_bucket;
    const uint32_t g = blockIdx.x / per_group, j = blockIdx.x - g * per_group;
    const uint32_t g0 = g * kApplyInterleave;
    if (g0 >= a.nb) return 0;
    const uint32_t gb = (a.nb - g0 < kApplyInterleave) ? (a.nb - g0) : kApplyInterleave;   // buckets in this group
    const uint32_t c = j / gb;
    b = g0 + (j - c * gb);
    if (b >= a.nb) return 0;
    const uint32_t cnt_true = a.counts[b];
    const uint64_t cnt = ((uint64_t)cnt_true < a.cap) ? cnt_true : a.cap;
    start = (uint64_t)c * kApplyChunk;
    if (start >= cnt) return 0;
    return (uint32_t)((cnt - start < kApplyChunk) ? (cnt - start) : kApplyChunk);
}

// Scatter of one thread's kApplyPer pairs of bucket b; pair j is live when bit j of `live` is set.  The stores carry
// the non-temporal hint: each lands in a line nothing else will touch soon, and measures 10 % faster that way.
// idx holds tensor-flat indices (single tensor) or positions inside the bucket (lists).  For lists the
// bucket's segment table is cached in LDS (start inside the bucket -> byte address of that element), and stays there for the
// workgroup's next chunk of the same bucket (fill = false).
template <bool MULTI, int EB = 2>
__device__ __forceinline__ void scatter_pairs(const ApplyArgs &a, ApplyShared &sh, uint32_t b,
                                              const int32_t (&idx)[kApplyPer], const uint16_t (&val)[kApplyPer],
                                              uint32_t live, bool fill = true) {
    typedef typename Elem<EB>::type T;       // width of a stored value; val[] holds it zero-extended
    bool bad = false;
    if (MULTI) {
        const uint64_t b0 = (uint64_t)b * a.be;
        const uint32_t blen = (uint32_t)((a.total - b0 < a.be) ? (a.total - b0) : a.be);
        const uint32_t s_lo = a.seg_begin[b], s_hi = a.seg_begin[b + 1];
        const uint32_t nseg = s_hi - s_lo;
        const bool cached = nseg <= kSegCache;                 // uniform
        if (cached && fill) {
            for (uint32_t s = threadIdx.x; s < nseg; s += kThreads) {
                const SegDesc d = a.segs[s_lo + s];
                sh.off[s] = d.bucket_off;
                // byte address of the element at bucket position 0 of this segment's tensor run
                sh.base[s] = (unsigned long long)(uintptr_t)a.wptrs[(uint64_t)d.tensor * (1u + a.wptr_skip)] +
                             (unsigned long long)EB * d.tensor_off -
                             (unsigned long long)EB * d.bucket_off;
            }
            if (threadIdx.x == 0) sh.off[nseg] = blen;
            __syncthreads();
        }
        uint32_t hint = 0;                                      // segment of the previous pair (payloads ascend)
#pragma unroll
        for (int j = 0; j < kApplyPer; ++j) {
            if (!((live >> j) & 1u)) continue;
            const uint32_t i = (uint32_t)idx[j];
            if (i >= blen) { bad = true; continue; }
            if (cached) {
                uint32_t lo = hint;
                if (!(sh.off[lo] <= i && i < sh.off[lo + 1])) {
                    lo = 0; uint32_t hi = nseg;                 // off[lo] <= i < off[hi]
                    while (hi - lo > 1) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (sh.off[mid] <= i) lo = mid; else hi = mid;
                    }
                    hint = lo;
                }
                __builtin_nontemporal_store((T)val[j], (gptr<T>)(uintptr_t)(sh.base[lo] + (unsigned long long)EB * i));
            } else {
                uint32_t lo = s_lo, hi = s_hi;                  // segs[lo].bucket_off <= i < segs[hi].bucket_off
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (a.segs[mid].bucket_off <= i) lo = mid; else hi = mid;
                }
                const SegDesc d = a.segs[lo];
                const uint32_t off = i - d.bucket_off;
                if (off >= d.len) { bad = true; continue; }     // cannot happen for a well-formed plan
                __builtin_nontemporal_store((T)val[j], (gptr<T>)a.wptrs[(uint64_t)d.tensor * (1u + a.wptr_skip)] +
                                                           ((uint64_t)d.tensor_off + off));
            }
        }
    } else {
        const uint64_t lo = (uint64_t)b * a.be;
        const uint64_t hi = (lo + a.be < a.n) ? (lo + a.be) : a.n;
#pragma unroll
        for (int j = 0; j < kApplyPer; ++j) {
            if (!((live >> j) & 1u)) continue;
            const int64_t i = idx[j];
            if (i < (int64_t)lo || i >= (int64_t)hi) { bad = true; continue; }
            __builtin_nontemporal_store((T)val[j], (gptr<T>)a.w + i);
        }
    }
    if (bad) atomicOr(a.flags, kFlagBadIndex);
}

// 32-bit indices
template <bool MULTI, int EB>
__device__ __forceinline__ void apply_pairs(const ApplyArgs &a, ApplyShared &sh, uint32_t b, uint64_t start, uint32_t nvalid,
                                            bool fill = true) {
    typedef typename Elem<EB>::type T;
    const int32_t *const Ib = a.I + (uint64_t)b * a.cap + start;
    const T *const Vb = reinterpret_cast<const T *>(a.V) + (uint64_t)b * a.cap + start;
    int32_t idx[kApplyPer];
    uint16_t val[kApplyPer];
    uint32_t live = 0;
#pragma unroll
    for (int j = 0; j < kApplyPer; ++j) {           // pair k = thread + j*256: contiguous per wave
        const uint32_t k = threadIdx.x + j * kThreads;
        const bool ok = k < nvalid;
        idx[j] = ok ? Ib[k] : 0;
        val[j] = ok ? Vb[k] : (uint16_t)0;
        live |= ok ? (1u << j) : 0u;
    }
    scatter_pairs<MULTI, EB>(a, sh, b, idx, val, live, fill);
}

template <bool MULTI, int EB = 2>
__global__ __launch_bounds__(kThreads) void apply_kernel(const ApplyArgs a) {
    __shared__ ApplyShared sh;
    uint32_t b; uint64_t start;
    const uint32_t nvalid = apply_chunk(a, a.chunks_per_bucket, b, start);
    if (nvalid == 0) return;
    apply_pairs<MULTI, EB>(a, sh, b, start, nvalid);
}

// The same for payloads whose slots are as large as their buckets (a caller that does not know the density): nearly all
// slots are empty then, and the workgroups that find nothing, 0.43 ns each, bound the launch (400 M slots in one bucket, 0.05 %
// changed: 85 us, 13.5 here).  The first `direct` chunks of each bucket keep a workgroup of their own, in
// apply_kernel's order; behind them a workgroup takes `group` chunks of one bucket in a row and fills the segment cache once.
template <bool MULTI, int EB = 2>
__global__ __launch_bounds__(kThreads) void apply_grouped_kernel(const ApplyArgs a) {
    __shared__ ApplyShared sh;
    uint32_t b; uint64_t start;
    const uint32_t singles = a.direct * a.nb;
    if (blockIdx.x < singles) {
        const uint32_t nvalid = apply_chunk(a, a.direct, b, start);
        if (nvalid) apply_pairs<MULTI, EB>(a, sh, b, start, nvalid);
        return;
    }
    const uint32_t t = blockIdx.x - singles, g = t / a.nb;
    b = t - g * a.nb;
    const uint32_t first = a.direct + g * a.group;
    const uint32_t end = (first + a.group < a.chunks_per_bucket) ? first + a.group : a.chunks_per_bucket;
    const uint32_t cnt_true = a.counts[b];
    uint64_t stop = (uint64_t)end * kApplyChunk;
    if ((uint64_t)cnt_true < stop) stop = cnt_true;
    if (a.cap < stop) stop = a.cap;
    start = (uint64_t)first * kApplyChunk;
    for (bool fill = true; start < stop; start += kApplyChunk, fill = false) {
        const uint64_t left = stop - start;
        apply_pairs<MULTI, EB>(a, sh, b, start, (uint32_t)(left < kApplyChunk ? left : kApplyChunk), fill);
    }
}

// The per-tensor view of a list payload: Alg. 2's message carries, per parameter tensor, int32 indices into that
// tensor's flattened elements; pair r of bucket b is at packed position b*be + I, inside exactly one segment of the
// bucket.  tensor_id / tensor_idx are laid out like I.  Same workgroup-to-chunk mapping and segment search as apply.
__global__ __launch_bounds__(kThreads) void tensor_view_kernel(const ApplyArgs a, uint32_t *tensor_id, int32_t *tensor_idx) {
    uint32_t b; uint64_t start;
    const uint32_t nvalid = apply_chunk(a, a.chunks_per_bucket, b, start);
    if (nvalid == 0) return;
    const uint64_t b0 = (uint64_t)b * a.be;
    const uint32_t blen = (uint32_t)((a.total - b0 < a.be) ? (a.total - b0) : a.be);
    const uint32_t s_lo = a.seg_begin[b], s_hi = a.seg_begin[b + 1];
    const uint64_t row = (uint64_t)b * a.cap + start;
    bool bad = false;
    for (uint32_t k = threadIdx.x; k < nvalid; k += kThreads) {
        const int32_t iv = a.I[row + k];
        if (iv < 0 || (uint32_t)iv >= blen) { bad = true; continue; }
        const uint32_t i = (uint32_t)iv;
        uint32_t lo = s_lo, hi = s_hi;                  // segs[lo].bucket_off <= i < segs[hi].bucket_off
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (a.segs[mid].bucket_off <= i) lo = mid; else hi = mid;
        }
        const SegDesc d = a.segs[lo];
        const uint32_t off = i - d.bucket_off;
        if (off >= d.len) { bad = true; continue; }     // cannot happen for a well-formed plan
        tensor_id[row + k] = d.tensor;
        tensor_idx[row + k] = (int32_t)(d.tensor_off + off);
    }
    if (bad) atomicOr(a.flags, kFlagBadIndex);
}

// 16-bit first differences (Sec. 3.3, index delta coding) decoded on the fly: thread t loads the
// kApplyPer consecutive differences t*8 .. t*8+7 of the chunk and sums them, the workgroup scans the
// 256 thread sums (DPP wave scan + LDS), and the chunk's anchor (the position of its first pair) turns
// the running sums into positions inside the bucket.  The positions then change hands through LDS so that
// thread t scatters pairs t, t+256, ...: one store instruction of a wave covers 64 consecutive pairs (about 13 KB
// of weights at 1 % density) as in apply_kernel, not every eighth pair of 512 (100 KB), which takes the memory
// side half as long again (12.4 against 8.2 ms on the 910-bucket benchmark set).  Buckets with differences that do not fit
// are scattered from their 32-bit indices by the same launch (by a second one before: values of 64 buckets of 335 k pairs
// decoded and applied 777 us, 770 now; of one bucket of 2.6 k pairs 28.6 / 27.2)
template <bool MULTI>
__global__ __launch_bounds__(kThreads) void apply_encoded_kernel(const ApplyArgs a) {
    __shared__ ApplyShared sh;
    __shared__ int32_t s_pos[kApplyChunk + kApplyChunk / 8];    // pair k at k + k/8: both access patterns spread over the banks
    uint32_t b; uint64_t start;
    const uint32_t nvalid = apply_chunk(a, a.chunks_per_bucket, b, start);
    if (nvalid == 0) return;
    if (a.max_gap[b] >= kWideGap) {                 // uniform: this bucket travels with 32-bit indices
        apply_pairs<MULTI, 2>(a, sh, b, start, nvalid);
        return;
    }
    const uint16_t *const Db = a.D + (uint64_t)b * a.cap + start;
    const uint16_t *const Vb = a.V + (uint64_t)b * a.cap + start;
    const uint32_t k0 = threadIdx.x * kApplyPer;
    static_assert(kApplyPer == 8, "one 16-byte vector of differences per thread");
    uint32_t d[kApplyPer];
    if ((((uintptr_t)Db) & 15u) == 0 && k0 + kApplyPer <= nvalid) {
        const u32x4 dv = *reinterpret_cast<const u32x4 *>(Db + k0);
#pragma unroll
        for (int j = 0; j < kApplyPer; ++j) d[j] = pattern_at(dv, j);
    } else {
#pragma unroll
        for (int j = 0; j < kApplyPer; ++j) d[j] = (k0 + j < nvalid) ? (uint32_t)Db[k0 + j] : 0u;
    }
    uint16_t val[kApplyPer];
    uint32_t live = 0;
#pragma unroll
    for (int j = 0; j < kApplyPer; ++j) {            // the values of the pairs this thread will scatter
        const uint32_t k = threadIdx.x + j * kThreads;
        const bool ok = k < nvalid;
        val[j] = ok ? Vb[k] : (uint16_t)0;
        live |= ok ? (1u << j) : 0u;
    }
    const uint32_t first = Db[0];                    // the chunk's first difference is covered by the anchor
    uint32_t run = 0;
#pragma unroll
    for (int j = 0; j < kApplyPer; ++j) { run += d[j]; d[j] = run; }      // inclusive inside the thread
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t inc = wave_inclusive_scan(run);
    if (lane == 63) sh.wave_total[wave] = inc;
    __syncthreads();
    uint32_t before = inc - run;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) before += (w < wave) ? sh.wave_total[w] : 0u;
    const uint32_t nchunk = a.chunks_per_bucket;
    const int32_t anchor = a.anchors[(uint64_t)b * nchunk + (uint32_t)(start / kApplyChunk)];
    const int64_t origin = (int64_t)anchor - (int64_t)first + (int64_t)((uint64_t)b * a.base_stride);
#pragma unroll
    for (int j = 0; j < kApplyPer; ++j) s_pos[k0 + j + threadIdx.x] = (int32_t)(origin + (int64_t)before + (int64_t)d[j]);
    __syncthreads();
    int32_t idx[kApplyPer];
#pragma unroll
    for (int j = 0; j < kApplyPer; ++j) {
        const uint32_t k = threadIdx.x + j * kThreads;
        idx[j] = s_pos[k + (k >> 3)];
    }
    scatter_pairs<MULTI>(a, sh, b, idx, val, live);
}

// First differences of each bucket's ascending indices, the bucket's largest difference and the
// anchors (position of the first pair of every chunk of kApplyChunk pairs).  Indices that do not ascend raise kFlagBadIndex and
// force the bucket to 32-bit transport.
// The largest difference of each chunk goes to gaps, from where max_gap_kernel takes those of the buckets; where there is no room
// for it (gaps null) to max_gap by atomics, which must be zero on entry then.  The words of all buckets lie in a few cache
// lines, where atomics take turns of 11 ns.  The differences are stored past the caches, which keeps the values that are coded
// next in them.  By atomics and with ordinary stores / as it is, us: 240 buckets of 335 k pairs 99 / 91 (and the coding of their
// values 104 / 101), 60 of them 54 / 24, 8 of 1 M 52 / 12, 20 of 250 k 29 / 9.
__global__ __launch_bounds__(kThreads) void encode_indices_kernel(const ApplyArgs a, uint16_t *D, uint32_t *max_gap,
                                                                  int32_t *anchors, uint32_t *gaps) {
    __shared__ uint32_t s_gap[kWaves];
    uint32_t b; uint64_t start;
    const uint32_t nvalid = apply_chunk(a, a.chunks_per_bucket, b, start);
    if (nvalid == 0) return;
    const int32_t *const Ib = a.I + (uint64_t)b * a.cap;
    const int64_t base = (int64_t)((uint64_t)b * a.base_stride);
    uint32_t gap = 0;
    bool bad = false;
    uint16_t *const Db = D + (uint64_t)b * a.cap;
    const uint32_t k0 = threadIdx.x * kApplyPer;
    static_assert(kApplyPer == 8, "eight consecutive pairs per thread: two 16-byte loads, one 16-byte store");
    // cap is a multiple of 4 whenever the rows of I are 16-byte aligned for every bucket; checked on the addresses
    const bool vec = (((uintptr_t)(Ib + start) | (uintptr_t)(Db + start)) & 15u) == 0;       // uniform over the workgroup
    if (vec && k0 + kApplyPer <= nvalid) {
        const uint64_t r0 = start + k0;
        const u32x4 lo = *reinterpret_cast<const u32x4 *>(Ib + r0), hi = *reinterpret_cast<const u32x4 *>(Ib + r0 + 4);
        const int32_t idx[8] = {(int32_t)lo.x, (int32_t)lo.y, (int32_t)lo.z, (int32_t)lo.w,
                                (int32_t)hi.x, (int32_t)hi.y, (int32_t)hi.z, (int32_t)hi.w};
        int64_t prev = r0 ? ((int64_t)Ib[r0 - 1] - base) : 0;
        uint32_t d16[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t cur = (int64_t)idx[j] - base;
            int64_t dd = cur - prev;
            if (dd < 0 || cur < 0) { bad = true; dd = 0xFFFFFFFFll; }
            d16[j] = (uint32_t)((uint64_t)dd & 0xFFFFu);
            gap = ((uint64_t)dd > gap) ? (uint32_t)dd : gap;
            prev = cur;
        }
        u32x4 out;
        out.x = d16[0] | (d16[1] << 16); out.y = d16[2] | (d16[3] << 16);
        out.z = d16[4] | (d16[5] << 16); out.w = d16[6] | (d16[7] << 16);
        store16_nt(as_global((void *)(Db + r0)), out);
        if (k0 == 0) anchors[(uint64_t)b * a.chunks_per_bucket + (uint32_t)(start / kApplyChunk)] = (int32_t)((int64_t)idx[0] - base);
    } else {
#pragma unroll
        for (int j = 0; j < kApplyPer; ++j) {            // the chunk's ragged end, or rows that are not 16-byte aligned
            const uint32_t k = vec ? (k0 + j) : (threadIdx.x + j * kThreads);
            if (k >= nvalid) continue;
            const uint64_t r = start + k;
            const int64_t cur = (int64_t)Ib[r] - base;
            const int64_t prev = r ? ((int64_t)Ib[r - 1] - base) : 0;
            int64_t dd = cur - prev;
            if (dd < 0 || cur < 0) { bad = true; dd = 0xFFFFFFFFll; }
            Db[r] = (uint16_t)((uint64_t)dd & 0xFFFFu);
            gap = ((uint64_t)dd > gap) ? (uint32_t)dd : gap;
            if (k == 0) anchors[(uint64_t)b * a.chunks_per_bucket + (uint32_t)(start / kApplyChunk)] = (int32_t)cur;
        }
    }
    // workgroup maximum: wave maximum by DPP-free shuffles is overkill here; use LDS atomics
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) s_gap[wave] = 0;
    __syncthreads();
    if (gap) atomicMax(&s_gap[wave], gap);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t g = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) g = s_gap[w] > g ? s_gap[w] : g;
        if (gaps) gaps[(uint64_t)b * a.chunks_per_bucket + (uint32_t)(start / kApplyChunk)] = g;
        else if (g) atomicMax(max_gap + b, g);
    }
    if (bad) atomicOr(a.flags, kFlagBadIndex);
}

// max_gap[b]: the largest difference of bucket b, from those of its chunks.  One wave per bucket.
__global__ __launch_bounds__(64) void max_gap_kernel(const uint32_t *gaps, const uint32_t *counts, uint64_t cap, uint32_t chunks_per_bucket,
                                                     uint32_t *max_gap) {
    const uint32_t b = blockIdx.x;
    const uint64_t cnt = ((uint64_t)counts[b] < cap) ? counts[b] : cap;
    const uint32_t live = (uint32_t)((cnt + kApplyChunk - 1) / kApplyChunk);
    uint32_t g = 0;
    for (uint32_t c = threadIdx.x; c < live; c += 64) {
        const uint32_t x = gaps[(uint64_t)b * chunks_per_bucket + c];
        g = x > g ? x : g;
    }
#pragma unroll
    for (int m = 32; m; m >>= 1) {
        const uint32_t x = (uint32_t)__shfl_xor((int)g, m, 64);
        g = x > g ? x : g;
    }
    if (threadIdx.x == 0) max_gap[b] = g;
}

// ---------------------------------------------------------------------------------------------
// density routing (Sec. 3.4): buckets whose sparse payload would not be smaller than their dense bytes,
// or that overflowed their slot, travel as a full copy.
// ---------------------------------------------------------------------------------------------
struct RouteArgs {
    const uint32_t *counts; uint32_t nb; uint64_t be; uint64_t total; uint64_t cap;
    uint32_t bytes_per_pair; uint32_t max_dense;
    int32_t *route_slot; uint32_t *sparse_counts; int32_t *dense_bucket; uint32_t *n_dense;
    uint32_t *flags;
};

// One workgroup walks the buckets 256 at a time, so that dense slots are handed out in bucket order.
__global__ __launch_bounds__(kThreads) void route_kernel(const RouteArgs a) {
    __shared__ uint32_t s_wave[kWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t taken = 0;                                 // dense buckets before this round (uniform)
    bool dropped = false;
    for (uint32_t b0 = 0; b0 < a.nb; b0 += kThreads) {
        const uint32_t b = b0 + threadIdx.x;
        bool dense = false;
        uint32_t cnt = 0;
        if (b < a.nb) {
            cnt = a.counts[b];
            const uint64_t lo = (uint64_t)b * a.be;
            const uint64_t len = (lo + a.be < a.total) ? a.be : (a.total > lo ? a.total - lo : 0);
            dense = ((uint64_t)cnt > a.cap) || (cnt > 0 && (uint64_t)cnt * a.bytes_per_pair >= 2 * len);
        }
        const unsigned long long mask = __ballot(dense);
        const uint32_t in_wave = __builtin_popcountll(mask & ((1ull << lane) - 1ull));
        if (lane == 0) s_wave[wave] = (uint32_t)__builtin_popcountll(mask);
        __syncthreads();
        uint32_t before = taken, round_total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { before += (w < wave) ? s_wave[w] : 0u; round_total += s_wave[w]; }
        __syncthreads();
        if (b < a.nb) {
            const uint32_t slot = before + in_wave;
            if (dense && slot < a.max_dense) {
                a.route_slot[b] = (int32_t)slot; a.dense_bucket[slot] = (int32_t)b; a.sparse_counts[b] = 0;
            } else {
                if (dense) dropped = true;
                a.route_slot[b] = -1;
                a.sparse_counts[b] = ((uint64_t)cnt < a.cap) ? cnt : (uint32_t)a.cap;
            }
        }
        taken += round_total;
    }
    if (threadIdx.x == 0) *a.n_dense = (taken < a.max_dense) ? taken : a.max_dense;
    if (dropped) atomicOr(a.flags, kFlagOverflow);
}

struct DenseCopyArgs {
    const TileDesc *tiles; const uint32_t *bucket_first; const PtrPair *pairs; uint16_t *const *wptrs;
    const int32_t *dense_bucket; const uint32_t *n_dense; uint32_t max_dense; uint32_t tiles_per_bucket_max;
    uint64_t be; uint16_t *dense;
};

// A workgroup copies len elements, source and destination each of any alignment: aligned 16-byte stores, kCopyLoads 16-byte
// loads per thread (at any address) in flight before the first of them, and single elements at the two ends.  Bound by
// memory.  Routed update of 300 odd-sized tensors end to end, new weights six bytes off (108 M elements, a fourth of the
// tensors changed by half): 533 us when runs that were not aligned on both sides were copied element by element, 238 us
// now; aligned runs (2 x 0.77 ms of the 3.0 ms of three 32B-shaped layers) are copied as fast as before.
constexpr int kCopyLoads = 4;

template <class T>
__device__ __forceinline__ void copy_run(gptr<T> dst, gptr<const T> src, uint32_t len) {
    constexpr uint32_t VE = 16u / sizeof(T);
    const uint32_t front = ((0u - (uint32_t)(uintptr_t)dst) & 15u) / (uint32_t)sizeof(T);
    const uint32_t lead = front < len ? front : len;
    const uint32_t nvec = (len - lead) / VE;
    if (threadIdx.x < lead) dst[threadIdx.x] = src[threadIdx.x];
    uint32_t v = threadIdx.x;
    for (; v + (kCopyLoads - 1) * kThreads < nvec; v += kCopyLoads * kThreads) {
        u32x4 x[kCopyLoads];
#pragma unroll
        for (int q = 0; q < kCopyLoads; ++q) x[q] = load16_any<true>(src + lead + (v + q * kThreads) * VE);
#pragma unroll
        for (int q = 0; q < kCopyLoads; ++q) store16_nt(dst + lead + (v + q * kThreads) * VE, x[q]);
    }
    for (; v < nvec; v += kThreads) store16_nt(dst + lead + v * VE, load16_any<true>(src + lead + v * VE));
    const uint32_t e = lead + nvec * VE + threadIdx.x;                 // fewer than VE are left
    if (e < len) dst[e] = src[e];
}

// PACK: dense[s] <- the new weights of bucket dense_bucket[s];  !PACK: resident weights <- dense[s].
// One workgroup per (dense slot, tile of the bucket), tiles as in extract's plan.
template <bool PACK>
__global__ __launch_bounds__(kThreads) void dense_copy_kernel(const DenseCopyArgs a) {
    const uint32_t s = blockIdx.x / a.tiles_per_bucket_max;
    const uint32_t j = blockIdx.x - s * a.tiles_per_bucket_max;
    if (s >= a.max_dense || s >= *a.n_dense) return;
    const uint32_t b = (uint32_t)a.dense_bucket[s];
    const uint32_t first = a.bucket_first[b];
    if (j >= a.bucket_first[b + 1] - first) return;
    const TileDesc d = a.tiles[first + j];
    uint16_t *const slot = a.dense + (uint64_t)s * a.be + d.bucket_off;
    uint16_t *const w = PACK ? const_cast<uint16_t *>(static_cast<const uint16_t *>(a.pairs[d.tensor].new_w)) + d.tensor_off
                             : a.wptrs[d.tensor] + d.tensor_off;
    const gptr<uint16_t> dst = as_global(PACK ? slot : w);
    const gptr<const uint16_t> src = as_global(static_cast<const uint16_t *>(PACK ? w : slot));
    copy_run<uint16_t>(dst, src, d.len);
}

// Second-pass snapshot refresh (Alg. 1's W_prev <- W done after the scan instead of inside it): the payload is
// scattered into the snapshot by apply_kernel, which cannot bring a bucket up to date whose payload was cut at cap.
// Those buckets are copied whole here.  kOverflowSplit workgroups per bucket walk its tiles (the plan's for a list,
// runs of tile_elems for a single tensor); a bucket that did not overflow costs one load of its count.
constexpr uint32_t kOverflowSplit = 16;

template <bool MULTI, int EB>
__global__ __launch_bounds__(kThreads) void refresh_overflow_kernel(const ExtractArgs a, uint32_t tile_elems) {
    typedef typename Elem<EB>::type T;
    const uint32_t b = blockIdx.x / kOverflowSplit, s = blockIdx.x - b * kOverflowSplit;
    if (b >= a.nb || (uint64_t)a.counts[b] <= a.cap) return;           // uniform over the workgroup
    uint64_t b0 = 0; uint32_t blen = 0, first = 0, nt;
    if (MULTI) {
        first = a.bucket_first[b];
        nt = a.bucket_first[b + 1] - first;
    } else {
        b0 = (uint64_t)b * a.be;
        blen = (uint32_t)((a.n - b0 < a.be) ? (a.n - b0) : a.be);
        nt = (blen + tile_elems - 1) / tile_elems;
    }
    for (uint32_t j = s; j < nt; j += kOverflowSplit) {
        gptr<T> dst; gptr<const T> src; uint32_t len;
        if (MULTI) {
            const TileDesc d = a.tiles[first + j];
            const PtrPair p = a.ptrs[d.tensor];
            dst = (gptr<T>)p.old_w + d.tensor_off;
            src = (gptr<const T>)as_global(p.new_w) + d.tensor_off;
            len = d.len;
        } else {
            const uint32_t off = j * tile_elems;
            len = (blen - off < tile_elems) ? (blen - off) : tile_elems;
            dst = (gptr<T>)a.old_w + b0 + off;
            src = (gptr<const T>)as_global(a.new_w) + b0 + off;
        }
        copy_run<T>(dst, src, len);
    }
}

// ---------------------------------------------------------------------------------------------
// value entropy coding (Sec. 3.3): static Huffman code over the high bytes of one bucket's values, low
// bytes raw.  Chunks of 2048 values, each chunk's bit stream in a slot of its own, a bit offset every 64
// values so that 32 lanes decode a chunk side by side.  Layout and code construction are those of the
// library header; the bit order is: most significant code bit first, stream bit i = bit (i & 31) of word i >> 5.
// ---------------------------------------------------------------------------------------------
constexpr uint32_t kVcChunk = 2048, kVcSlotWords = 768, kVcSub = 64, kVcMaxLen = 12;

struct ValueCodecArgs {
    const uint16_t *V; uint16_t *V_out; const uint32_t *counts; uint32_t nb; uint64_t cap; uint32_t nchunk;
    uint8_t *lens; uint8_t *low; uint32_t *bits; uint32_t *chunk_words; uint16_t *sub;
    uint32_t *hist;        // [nb*256] scratch, all 0 between calls
    uint32_t *rcode;       // [nb*256] scratch: bit-reversed canonical code of each symbol
    uint32_t *flags;
};

// per (bucket, chunk): histogram of the high bytes, accumulated per bucket
constexpr uint32_t kVcHistChunks = 8;        // chunks of one bucket counted by one workgroup

__global__ __launch_bounds__(kThreads) void vc_hist_kernel(const ValueCodecArgs a) {
    // The high bytes of a payload crowd into a handful of bins, and LDS atomics of one wave on one word take turns: every
    // two lanes count in a histogram of their own, with four bins to a word (two threads count 128 values, so a
    // byte holds any count), 65 words apart so that the same word of different histograms lies in different banks.
    // 240 buckets of 335 k values: 86 us with a 32-bit histogram per 8 lanes, 44 us now.
    constexpr uint32_t kParts = kThreads / 2, kPitch = 65;
    static_assert(kVcHistChunks * kVcChunk / kParts < 256u, "a byte holds every count of two threads");
    static_assert(kParts * kPitch % 4 == 0, "cleared in 16-byte stores");
    static_assert(kVcHistChunks * kVcChunk / kWaves < 65536u, "16 bits hold what a wave adds up");
    __shared__ __align__(16) uint32_t h[kParts * kPitch];
    __shared__ uint32_t s_sum[256];
    const uint32_t groups = (a.nchunk + kVcHistChunks - 1) / kVcHistChunks;
    const uint32_t b = blockIdx.x / groups, g = blockIdx.x - b * groups;
    const uint64_t cnt = ((uint64_t)a.counts[b] < a.cap) ? a.counts[b] : a.cap;
    const uint64_t g0 = (uint64_t)g * kVcHistChunks * kVcChunk;
    if (g0 >= cnt) return;
    const uint32_t s = threadIdx.x;
    uint32_t *const mine = h + (s >> 1) * kPitch;
    auto count = [&](uint32_t bin) { atomicAdd(&mine[bin >> 2], 1u << (8u * (bin & 3u))); };
    const uint32_t gn = (uint32_t)((cnt - g0 < (uint64_t)kVcHistChunks * kVcChunk) ? (cnt - g0) : kVcHistChunks * kVcChunk);
    const u32x4 zero = {0, 0, 0, 0};
    for (uint32_t i = s; i < kParts * kPitch / 4; i += kThreads) reinterpret_cast<u32x4 *>(h)[i] = zero;
    s_sum[s] = 0;
    __syncthreads();
    const uint16_t *v = a.V + (uint64_t)b * a.cap + g0;
    if ((((uintptr_t)v) & 15u) == 0) {
        constexpr uint32_t kSteps = kVcHistChunks * kVcChunk / (8 * kThreads);   // 8 values per 16-byte load
        u32x4 x[kSteps];
        const u32x4 none = {0, 0, 0, 0};
#pragma unroll
        for (uint32_t q = 0; q < kSteps; ++q) {
            const uint32_t i0 = (q * kThreads + s) * 8u;
            x[q] = (i0 + 8u <= gn) ? *reinterpret_cast<const u32x4 *>(v + i0) : none;
        }
#pragma unroll
        for (uint32_t q = 0; q < kSteps; ++q) {
            const uint32_t i0 = (q * kThreads + s) * 8u;
            if (i0 + 8u <= gn) {
                const uint32_t d[4] = {x[q].x, x[q].y, x[q].z, x[q].w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    count((d[c] >> 8) & 0xFFu);
                    count(d[c] >> 24);
                }
            } else {
                for (uint32_t i = i0; i < gn; ++i) count(v[i] >> 8);
            }
        }
    } else {
        for (uint32_t i = s; i < gn; i += kThreads) count(v[i] >> 8);
    }
    __syncthreads();
    // every wave adds up a quarter of the histograms, a lane one word of them, two bins to a 16-bit field each
    const uint32_t word = s & 63u, p0 = (s >> 6) * (kParts / kWaves);
    uint32_t even = 0, odd = 0;
#pragma unroll 8
    for (uint32_t p = 0; p < kParts / kWaves; ++p) {
        const uint32_t x = h[(p0 + p) * kPitch + word];
        even += x & 0x00FF00FFu;
        odd += (x >> 8) & 0x00FF00FFu;
    }
    const uint32_t n[4] = {even & 0xFFFFu, odd & 0xFFFFu, even >> 16, odd >> 16};
#pragma unroll
    for (uint32_t c = 0; c < 4; ++c)
        if (n[c]) atomicAdd(&s_sum[4u * word + c], n[c]);
    __syncthreads();
    if (s_sum[s]) atomicAdd(a.hist + (uint64_t)b * 256 + s, s_sum[s]);
}

// One workgroup per bucket builds the Huffman lengths exactly as the header specifies (merge the two smallest
// live nodes, ties to the smaller id; weights halved until no length exceeds 12), then all threads derive the
// canonical codes.  Node ids 0..255 are the symbols, 256.. the merged nodes in order of creation.  The symbols are sorted
// once by (weight, id); merged nodes come into being in ascending (weight, id) order by themselves, so the two
// smallest live nodes are always at the heads of these two queues, and a tie between them goes to the symbol.  One wave
// runs the merge with both queues in registers and the queue heads in scalar registers: a step is a few readlanes.  Up
// to kVcWave symbols (the high bytes of weights are 20 to 30) a wave also sorts and measures the depths by itself, and the
// four or eight waves try successive halvings side by side; more symbols take R = 4 registers per lane and queue (entry i in lane i & 63
// of register i >> 6) and the whole workgroup around the merge.  Bound by the serial chain.  240 buckets of 335 k
// values: 147 us when every step searched all nodes for its two minima with 64-bit wave reductions, 49 us by the general
// path, 15 us with four waves (two tries of four).  The whole value coder with 4 / 8 / 16 waves, us: 240 buckets of 335 k values
// 101 / 95 / 97, 20 of 250 k 30 / 24 / 26, 8 of 1 M (eight halvings) 39 / 33 / 30, 240 of 10 k 23 / 22 / 24.
__device__ __forceinline__ uint32_t lane_value(uint32_t x, uint32_t lane) { return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)lane); }

__device__ __forceinline__ void vc_merge(uint32_t used, const uint32_t *sorted_w, const uint8_t *sorted_s, int16_t *parent, int lane) {
    constexpr int R = 4;                                     // 256 symbols, 64 lanes
    uint32_t leaf[R], node[R], leaf_up[R], node_up[R];       // weights; ids of the parents
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t i = (uint32_t)lane + 64u * r;
        leaf[r] = i < used ? sorted_w[i] : 0u;
        node[r] = leaf_up[r] = node_up[r] = 0u;
    }
    uint32_t nl = 0, nn = 0;                                 // heads of the two queues
    for (uint32_t made = 0; made + 1 < used; ++made) {       // `made` is also the end of the queue of merged nodes
        uint32_t sum = 0;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            uint32_t wl = 0, wn = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if ((nl >> 6) == (uint32_t)r) wl = lane_value(leaf[r], nl & 63u);
                if ((nn >> 6) == (uint32_t)r) wn = lane_value(node[r], nn & 63u);
            }
            const bool take_leaf = nl < used && (nn >= made || wl <= wn);      // one of the two queues has an entry
            const uint32_t at = take_leaf ? nl : nn;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const bool here = (at >> 6) == (uint32_t)r && (at & 63u) == (uint32_t)lane;
                if (here && take_leaf) leaf_up[r] = 256u + made;
                if (here && !take_leaf) node_up[r] = 256u + made;
            }
            sum += take_leaf ? wl : wn;
            nl += take_leaf ? 1u : 0u;
            nn += take_leaf ? 0u : 1u;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if ((made >> 6) == (uint32_t)r && (made & 63u) == (uint32_t)lane) node[r] = sum;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {                            // the root has no parent: -1 stands
        const uint32_t i = (uint32_t)lane + 64u * r;
        if (i < used && leaf_up[r]) parent[sorted_s[i]] = (int16_t)leaf_up[r];
        if (i + 2 < used) parent[256 + i] = (int16_t)node_up[r];               // used - 1 merged nodes, the last is the root
    }
}

// Code length of symbol number `lane` of `used` = 2 .. kVcWave (weight w, 0 for lanes past the last; lanes in symbol order).
// perm: 64 words of LDS of this wave's own.  No branches inside a step: a queue that is empty shows the largest word.
constexpr uint32_t kVcWave = 63;

__device__ __forceinline__ uint32_t vc_wave_lengths(uint32_t w, uint32_t used, uint32_t *perm, int lane) {
    constexpr uint32_t kEmpty = 0xFFFFFFFFu;
    const uint32_t me = (uint32_t)lane;
    uint32_t rank = 0;                                       // by (weight, symbol)
    for (uint32_t i = 0; i < used; ++i) {
        const uint32_t x = lane_value(w, i);
        rank += (x < w || (x == w && i < me)) ? 1u : 0u;
    }
    if (me < used) perm[rank] = w;
    __builtin_amdgcn_wave_barrier();                         // one wave: its LDS operations stay in order
    const uint32_t leaf = me < used ? *(volatile uint32_t *)(perm + lane) : kEmpty;
    uint32_t node = kEmpty, up = 0, leaf_up = 0;             // merged weights, their parents, the sorted symbols' parents
    uint32_t nl = 0, nn = 0;                                 // at most 63 each
    for (uint32_t made = 0; made + 1 < used; ++made) {
        uint32_t sum = 0;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t wl = lane_value(leaf, nl), wn = lane_value(node, nn);
            const bool take_leaf = wl <= wn;
            leaf_up = me == (take_leaf ? nl : 64u) ? made : leaf_up;
            up = me == (take_leaf ? 64u : nn) ? made : up;
            sum += take_leaf ? wl : wn;
            nl += take_leaf ? 1u : 0u;
            nn += take_leaf ? 0u : 1u;
        }
        node = (me == made) ? sum : node;
    }
    uint32_t depth = 0;                                      // of the merged nodes, from the root down
    for (int k = (int)used - 3; k >= 0; --k) {
        const uint32_t d = lane_value(depth, lane_value(up, (uint32_t)k)) + 1u;
        depth = (lane == k) ? d : depth;
    }
    const uint32_t sorted_len = (uint32_t)__shfl((int)depth, (int)leaf_up, 64) + 1u;
    const uint32_t l = (uint32_t)__shfl((int)sorted_len, (int)(rank & 63u), 64);
    return me < used ? l : 0u;
}

// W waves; the first 256 threads hold a symbol each
template <int W>
__global__ __launch_bounds__(64 * W) void vc_build_kernel(const ValueCodecArgs a) {
    __shared__ int16_t parent[512];
    __shared__ __align__(16) uint32_t packed_w[256];         // weights of the symbols that occur, in symbol order, then 0
    __shared__ uint32_t sorted_w[64 * W];
    __shared__ uint8_t sorted_s[256];
    __shared__ uint32_t count_l[kVcMaxLen + 1][kWaves];
    __shared__ uint32_t s_used[kWaves], s_maxlen, s_fits[W];
    __shared__ uint8_t s_len[64 * W];
    const uint32_t b = blockIdx.x, s = threadIdx.x;
    const int lane = s & 63, wave = s >> 6;
    const bool symbol = s < 256;                             // uniform per wave
    uint32_t w = 0;
    if (symbol) {
        w = a.hist[(uint64_t)b * 256 + s];
        a.hist[(uint64_t)b * 256 + s] = 0;                   // as vc_hist_kernel finds it next time
        packed_w[s] = 0;
    }
    const unsigned long long there = __ballot(w != 0);
    if (symbol && lane == 0) s_used[wave] = (uint32_t)__builtin_popcountll(there);
    __syncthreads();
    uint32_t used = 0, place = (uint32_t)__builtin_popcountll(there & ((1ull << lane) - 1ull));
#pragma unroll
    for (int v = 0; v < kWaves; ++v) { place += (v < wave) ? s_used[v] : 0u; used += s_used[v]; }
    used = uniform(used);
    uint32_t l = 0;
    if (used == 1) {
        l = w ? 1u : 0u;
    } else if (used > 1 && used <= kVcWave) {                // uniform
        if (w) packed_w[place] = w;
        __syncthreads();
        // r halvings make ceil(w / 2^r): the waves try W numbers of halvings at a time (335 k values take 6)
        for (uint32_t r0 = 0;; r0 += W) {          // 31 halvings leave weights of 1 and lengths of 6 at most
            const uint32_t r = r0 + (uint32_t)wave;
            const uint32_t wr = (uint32_t)(((uint64_t)packed_w[lane] + (1ull << r) - 1ull) >> r);
            const uint32_t len = vc_wave_lengths(wr, used, sorted_w + 64 * wave, lane);
            s_len[64 * wave + lane] = (uint8_t)len;
            const bool fits = !__any(len > kVcMaxLen);
            if (lane == 0) s_fits[wave] = fits ? 1u : 0u;
            __syncthreads();
            uint32_t hit = W;
#pragma unroll
            for (int v = W - 1; v >= 0; --v) hit = s_fits[v] ? (uint32_t)v : hit;
            hit = uniform(hit);
            if (hit < W) { l = w ? (uint32_t)s_len[64 * hit + place] : 0u; break; }
            __syncthreads();                                 // everybody has read s_fits
        }
    }
    while (used > kVcWave) {                                 // uniform: every thread takes every barrier
        if (w) packed_w[place] = w;
        if (symbol) { parent[s] = -1; parent[s + 256] = -1; }
        if (s == 0) s_maxlen = 0;
        __syncthreads();
        if (w) {                                             // rank by (weight, symbol): every weight is non-zero
            uint32_t rank = 0;
            for (uint32_t i = 0; i < used; i += 4) {         // entries past the last are 0 ...
                const u32x4 x = *reinterpret_cast<const u32x4 *>(packed_w + i);
                const uint32_t xi[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) rank += (xi[c] < w || (xi[c] == w && i + c < place)) ? 1u : 0u;
            }
            rank -= ((used + 3u) & ~3u) - used;              // ... and counted as smaller
            sorted_w[rank] = w;
            sorted_s[rank] = (uint8_t)s;
        }
        __syncthreads();
        if (wave == 0) {
            vc_merge(used, sorted_w, sorted_s, parent, lane);
        }
        __syncthreads();
        l = 0;
        if (w) {
            for (int jn = (int)s; parent[jn] >= 0; jn = parent[jn]) ++l;
            atomicMax(&s_maxlen, l);
        }
        __syncthreads();
        if (s_maxlen <= kVcMaxLen) break;
        w = w ? (w + 1) / 2 : 0u;
        __syncthreads();                                     // everybody has read s_maxlen
    }
    // canonical code = first code of its length + number of smaller symbols of the same length
    uint32_t rank = 0;
    if (symbol) {
        a.lens[(uint64_t)b * 256 + s] = (uint8_t)l;
        for (uint32_t j = 1; j <= kVcMaxLen; ++j) {
            const unsigned long long m = __ballot(l == j);
            if (l == j) rank = (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull));
            if (lane == 0) count_l[j][wave] = (uint32_t)__builtin_popcountll(m);
        }
    }
    __syncthreads();
    if (!symbol) return;
    uint32_t first = 0, code = 0;
    for (uint32_t j = 1; j <= kVcMaxLen; ++j) {
        uint32_t cj = 0;
#pragma unroll
        for (int v = 0; v < kWaves; ++v) { cj += count_l[j][v]; if (j == l && v < wave) rank += count_l[j][v]; }
        if (j == l) first = code;
        code = (code + cj) << 1;
    }
    const uint32_t c = first + rank;
    a.rcode[(uint64_t)b * 256 + s] = l ? (__brev(c) >> (32 - l)) : 0u;
}

// per (bucket, group of kVcEncodeChunks chunks), chunk after chunk with the bucket's code table loaded once: codes of
// 8 consecutive values per thread, assembled in a 128-bit buffer, placed in the chunk's LDS bit array at the offset a
// workgroup scan of the bit counts gives, then stored coalesced
constexpr uint32_t kVcEncodeChunks = 4;

__global__ __launch_bounds__(kThreads) void vc_encode_kernel(const ValueCodecArgs a) {
    __shared__ uint32_t s_code[256];                 // bit-reversed code | length << 16
    __shared__ uint32_t s_words[kVcSlotWords + 4];
    __shared__ uint32_t s_wave[kWaves];
    const uint32_t groups = (a.nchunk + kVcEncodeChunks - 1) / kVcEncodeChunks;
    const uint32_t b = blockIdx.x / groups, g = blockIdx.x - b * groups;
    const uint64_t cnt = ((uint64_t)a.counts[b] < a.cap) ? a.counts[b] : a.cap;
    const uint32_t k_lo = g * kVcEncodeChunks;
    const uint32_t k_hi = (k_lo + kVcEncodeChunks < a.nchunk) ? (k_lo + kVcEncodeChunks) : a.nchunk;
    if ((uint64_t)k_lo * kVcChunk < cnt) {
        s_code[threadIdx.x] = a.rcode[(uint64_t)b * 256 + threadIdx.x] | ((uint32_t)a.lens[(uint64_t)b * 256 + threadIdx.x] << 16);
        __syncthreads();
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t k = k_lo; k < k_hi; ++k) {
        const uint64_t r0 = (uint64_t)k * kVcChunk;
        const uint64_t slot = (uint64_t)b * a.nchunk + k;
        if (r0 >= cnt) {                                 // uniform: a chunk without values
            if (threadIdx.x == 0) a.chunk_words[slot] = 0;
            continue;
        }
        const uint32_t n = (uint32_t)((cnt - r0 < kVcChunk) ? (cnt - r0) : kVcChunk);
        const uint16_t *v = a.V + (uint64_t)b * a.cap + r0;
        uint8_t *lo = a.low + (uint64_t)b * a.cap + r0;
        const uint32_t k0 = threadIdx.x * 8;
        // the thread's 8 values: one 16-byte load and one 8-byte store of the low bytes where the rows allow it
        uint32_t xs[8];
        const bool vec = (k0 + 8 <= n) && (((((uintptr_t)(v + k0)) & 15u) | (((uintptr_t)(lo + k0)) & 7u)) == 0);
        if (vec) {
            const u32x4 q = *reinterpret_cast<const u32x4 *>(v + k0);
            xs[0] = q.x & 0xFFFFu; xs[1] = q.x >> 16; xs[2] = q.y & 0xFFFFu; xs[3] = q.y >> 16;
            xs[4] = q.z & 0xFFFFu; xs[5] = q.z >> 16; xs[6] = q.w & 0xFFFFu; xs[7] = q.w >> 16;
            uint2 lb;
            lb.x = (xs[0] & 0xFFu) | ((xs[1] & 0xFFu) << 8) | ((xs[2] & 0xFFu) << 16) | ((xs[3] & 0xFFu) << 24);
            lb.y = (xs[4] & 0xFFu) | ((xs[5] & 0xFFu) << 8) | ((xs[6] & 0xFFu) << 16) | ((xs[7] & 0xFFu) << 24);
            __builtin_nontemporal_store(((unsigned long long)lb.y << 32) | lb.x, as_global(reinterpret_cast<unsigned long long *>(lo + k0)));
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                xs[j] = (k0 + j < n) ? (uint32_t)v[k0 + j] : 0u;
                if (k0 + j < n) lo[k0 + j] = (uint8_t)(xs[j] & 0xFFu);
            }
        }
        // two halves of four codes each (at most 48 bits per half), joined into a 128-bit buffer afterwards;
        // stream order = ascending bit index
        unsigned long long half[2] = {0, 0};
        uint32_t hbits[2] = {0, 0};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (k0 + j < n) {
                const uint32_t c = s_code[xs[j] >> 8];
                half[j >> 2] |= (unsigned long long)(c & 0xFFFFu) << hbits[j >> 2];
                hbits[j >> 2] += c >> 16;
            }
        }
        const uint32_t nbits = hbits[0] + hbits[1];
        const unsigned long long buf0 = half[0] | (half[1] << hbits[0]);                       // hbits[0] <= 48
        const unsigned long long buf1 = hbits[0] ? (half[1] >> (64 - hbits[0])) : 0ull;
        const uint32_t inc = wave_inclusive_scan(nbits);
        if (lane == 63) s_wave[wave] = inc;
        __syncthreads();                                // also: every thread is done with the previous chunk's s_words
        uint32_t start = inc - nbits, total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { start += (w < wave) ? s_wave[w] : 0u; total += s_wave[w]; }
        const uint32_t used = (total + 31) / 32;         // at most kVcSlotWords: 2048 codes of at most kVcMaxLen bits
        for (uint32_t i = threadIdx.x; i < used + 4; i += kThreads) s_words[i] = 0;     // what this chunk can touch
        __syncthreads();
        if ((threadIdx.x & 7) == 0 && k0 < n) a.sub[slot * 32 + (threadIdx.x >> 3)] = (uint16_t)start;
        if (nbits) {
            const uint32_t w = start >> 5, sh = start & 31;
            // the thread's bits shifted to their place: up to 96 + 31 bits -> four words
            const uint32_t p0 = (uint32_t)buf0, p1 = (uint32_t)(buf0 >> 32), p2 = (uint32_t)buf1, p3 = (uint32_t)(buf1 >> 32);
            atomicOr(&s_words[w], p0 << sh);
            atomicOr(&s_words[w + 1], sh ? ((p0 >> (32 - sh)) | (p1 << sh)) : p1);
            atomicOr(&s_words[w + 2], sh ? ((p1 >> (32 - sh)) | (p2 << sh)) : p2);
            atomicOr(&s_words[w + 3], sh ? ((p2 >> (32 - sh)) | (p3 << sh)) : p3);
            if (sh && (p3 >> (32 - sh))) atomicOr(&s_words[w + 4], p3 >> (32 - sh));
        }
        __syncthreads();
        uint32_t *out = a.bits + slot * kVcSlotWords;
        for (uint32_t i = threadIdx.x; i < used; i += kThreads) __builtin_nontemporal_store(s_words[i], as_global(out + i));
        if (threadIdx.x == 0) a.chunk_words[slot] = used;
    }
}

// per (bucket, group of kVcDecodeChunks chunks): rebuild the code from its lengths, fill a 4096-entry table
// indexed by the next 12 stream bits, bring the group's bit streams into LDS, then all 256 threads decode at
// once -- 32 threads per chunk, 64 values each, every thread starting at its own recorded bit offset -- and the
// values (decoded high byte | stored low byte) are written coalesced
constexpr uint32_t kVcDecodeChunks = 8;
static_assert(kVcDecodeChunks * 32 == kThreads, "one thread per sub-block of the group");

__global__ __launch_bounds__(kThreads) void vc_decode_kernel(const ValueCodecArgs a) {
    __shared__ uint16_t s_lut[1u << kVcMaxLen];      // symbol << 4 | length
    __shared__ uint32_t s_cnt[kVcMaxLen + 1][kWaves];
    __shared__ uint8_t s_sorted[256];                // symbols in (length, symbol) order
    __shared__ uint32_t s_first[kVcMaxLen + 2], s_off[kVcMaxLen + 2];   // per length: first code, start in s_sorted
    __shared__ uint32_t s_words[kVcDecodeChunks][kVcSlotWords + 1];
    // decoded high bytes: value q*4 + c of thread t is byte c of word q * kSymPitch + t (the odd pitch keeps both
    // the decoders' stores and the write-out's loads off each other's LDS banks)
    constexpr uint32_t kSymPitch = kThreads + 1;
    __shared__ uint32_t s_sym[(kVcSub / 4) * kSymPitch];
    const uint32_t groups = (a.nchunk + kVcDecodeChunks - 1) / kVcDecodeChunks;
    const uint32_t b = blockIdx.x / groups, g = blockIdx.x - b * groups;
    const uint64_t cnt = ((uint64_t)a.counts[b] < a.cap) ? a.counts[b] : a.cap;
    const uint64_t g0 = (uint64_t)g * kVcDecodeChunks * kVcChunk;        // first value of the group
    if (g0 >= cnt) return;
    const uint32_t s = threadIdx.x;
    const int lane = s & 63, wave = s >> 6;
    uint32_t l = a.lens[(uint64_t)b * 256 + s];
    if (l > kVcMaxLen) l = 0;                        // not a length this format can hold: treated as absent
    // canonical code of symbol s = first code of its length + number of smaller symbols of that length
    uint32_t rank = 0;
    for (uint32_t j = 1; j <= kVcMaxLen; ++j) {
        const unsigned long long m = __ballot(l == j);
        if (l == j) rank = __builtin_popcountll(m & ((1ull << lane) - 1ull));
        if (lane == 0) s_cnt[j][wave] = (uint32_t)__builtin_popcountll(m);
    }
    // the group's streams: chunk kk of the group is chunk g*8 + kk of the bucket; chunks past the end read as empty
    const uint32_t gn = (uint32_t)((cnt - g0 < (uint64_t)kVcDecodeChunks * kVcChunk) ? (cnt - g0) : kVcDecodeChunks * kVcChunk);
    const uint32_t nch = (gn + kVcChunk - 1) / kVcChunk;                  // chunks of this group that hold values
    const uint64_t slot0 = (uint64_t)b * a.nchunk + (uint64_t)g * kVcDecodeChunks;
    {   // every load of the group's streams is issued before the first is stored (3 words per thread and chunk)
        static_assert(kVcSlotWords == 3 * kThreads, "three stream words per thread");
        uint32_t used[kVcDecodeChunks], tmp[kVcDecodeChunks][3];
#pragma unroll
        for (uint32_t kk = 0; kk < kVcDecodeChunks; ++kk) {
            used[kk] = (kk < nch) ? a.chunk_words[slot0 + kk] : 0u;
            used[kk] = used[kk] > kVcSlotWords ? kVcSlotWords : used[kk];
        }
#pragma unroll
        for (uint32_t kk = 0; kk < kVcDecodeChunks; ++kk) {
            const uint32_t *in = a.bits + (slot0 + kk) * kVcSlotWords;
#pragma unroll
            for (uint32_t r = 0; r < 3; ++r) tmp[kk][r] = (s + r * kThreads < used[kk]) ? in[s + r * kThreads] : 0u;
        }
#pragma unroll
        for (uint32_t kk = 0; kk < kVcDecodeChunks; ++kk) {
#pragma unroll
            for (uint32_t r = 0; r < 3; ++r) s_words[kk][s + r * kThreads] = tmp[kk][r];
        }
        if (s < kVcDecodeChunks) s_words[s][kVcSlotWords] = 0u;
    }
    __syncthreads();
    // Per length j: how many symbols have it, the first code of that length and where its symbols start in the
    // list of symbols sorted by (length, symbol) -- every thread keeps the three small tables in registers.
    // end_j[j]: one past the last code of length j, left-aligned to kVcMaxLen bits.  The runs of canonical codes of
    // the lengths 1, 2, ... follow one another in that space, so end_j never decreases.
    uint32_t off_j[kVcMaxLen + 1], end_j[kVcMaxLen + 1];
    {
        uint32_t code = 0, off = 0;
#pragma unroll
        for (uint32_t j = 1; j <= kVcMaxLen; ++j) {
            uint32_t cj = 0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) { cj += s_cnt[j][w]; if (j == l && w < wave) rank += s_cnt[j][w]; }
            off_j[j] = off; end_j[j] = (code + cj) << (kVcMaxLen - j);
            if (s == j) { s_first[j] = code; s_off[j] = off; }
            code = (code + cj) << 1; off += cj;
        }
        if (s == 0) { s_first[kVcMaxLen + 1] = 0; s_off[kVcMaxLen + 1] = 0; }
    }
#pragma unroll
    for (uint32_t j = 1; j <= kVcMaxLen; ++j)
        if (l == j) s_sorted[off_j[j] + rank] = (uint8_t)s;            // off + rank < 256: each symbol has one length
    __syncthreads();
    // Table entry i: the 12 stream bits i, first bit in bit 0, are a code word's bits most significant first;
    // the entry's length is the first length whose run ends above them (none: not a code of this table, entry 0).
    for (uint32_t i = s; i < (1u << kVcMaxLen); i += kThreads) {
        const uint32_t c12 = __brev(i) >> (32 - kVcMaxLen);
        uint32_t len = 1;
#pragma unroll
        for (uint32_t j = 1; j <= kVcMaxLen; ++j) len += (c12 >= end_j[j]) ? 1u : 0u;
        uint32_t e = 0;
        if (len <= kVcMaxLen) {
            const uint32_t d = (c12 >> (kVcMaxLen - len)) - s_first[len];      // below the count of that length
            e = ((uint32_t)s_sorted[(s_off[len] + d) & 255u] << 4) | len;
        }
        s_lut[i] = (uint16_t)e;
    }
    __syncthreads();
    bool bad = false;
    {
        const uint32_t kk = s >> 5, sb = s & 31u;                         // chunk of the group, sub-block of the chunk
        const uint32_t v0 = kk * kVcChunk + sb * kVcSub;                  // first value of this thread, inside the group
        if (v0 < gn) {
            const uint32_t v1 = (v0 + kVcSub < gn) ? (v0 + kVcSub) : gn;  // a chunk holds a multiple of kVcSub unless it is the last
            uint32_t pos = a.sub[(slot0 + kk) * 32 + sb];
            // one value: the next kVcMaxLen stream bits index the table.  A pattern that is no code of the table has
            // length 0: the position then stands still and the remaining values of the sub-block come out as that
            // entry's symbol -- the flag tells the caller that the output means nothing.  (The loop is bound by
            // instruction issue, so it carries no early exit and, for full sub-blocks, no per-value bookkeeping.)
            auto next = [&]() -> uint32_t {
                const uint32_t w = pos >> 5, sh = pos & 31;
                uint32_t x = 0;
                if (w < kVcSlotWords) x = (uint32_t)((((unsigned long long)s_words[kk][w + 1] << 32) | s_words[kk][w]) >> sh);
                const uint32_t e = s_lut[x & ((1u << kVcMaxLen) - 1u)];
                bad = bad || (e & 15u) == 0;
                pos += e & 15u;
                return e >> 4;
            };
            if (v1 - v0 == kVcSub) {
#pragma unroll 4
                for (uint32_t q = 0; q < kVcSub / 4; ++q) {
                    uint32_t pack = next();
                    pack |= next() << 8;
                    pack |= next() << 16;
                    pack |= next() << 24;
                    s_sym[q * kSymPitch + s] = pack;
                }
            } else {
                uint32_t pack = 0;
                for (uint32_t i = v0; i < v1; ++i) {
                    const uint32_t it = i - v0;
                    pack |= next() << (8u * (it & 3u));
                    if ((it & 3u) == 3u || i + 1 == v1) { s_sym[(it >> 2) * kSymPitch + s] = pack; pack = 0; }
                }
            }
        }
    }
    __syncthreads();
    const uint8_t *lo = a.low + (uint64_t)b * a.cap + g0;
    uint16_t *out = a.V_out + (uint64_t)b * a.cap + g0;
    if (((((uintptr_t)lo) & 7u) | (((uintptr_t)out) & 15u)) == 0) {
        // 8 consecutive values per thread and step: one 8-byte load of low bytes, two words of symbols, one
        // 16-byte store; all of a thread's loads are issued first
        constexpr uint32_t kSteps = kVcDecodeChunks * kVcChunk / (8 * kThreads);
        uint2 lw[kSteps];
#pragma unroll
        for (uint32_t q = 0; q < kSteps; ++q) {
            const uint32_t i0 = (q * kThreads + s) * 8u;
            lw[q] = (i0 + 8u <= gn) ? *reinterpret_cast<const uint2 *>(lo + i0) : make_uint2(0u, 0u);
        }
#pragma unroll
        for (uint32_t q = 0; q < kSteps; ++q) {
            const uint32_t i0 = (q * kThreads + s) * 8u;
            if (i0 + 8u <= gn) {
                const uint32_t t = i0 / kVcSub, w0 = (i0 % kVcSub) >> 2;
                const uint32_t lwq[2] = {lw[q].x, lw[q].y};
                uint32_t o[4];
#pragma unroll
                for (uint32_t c = 0; c < 2; ++c) {                        // 4 values per word of symbols / of low bytes
                    const uint32_t sy = s_sym[(w0 + c) * kSymPitch + t], lb = lwq[c];
                    o[2 * c] = ((sy & 0xFFu) << 8) | (lb & 0xFFu) | ((sy & 0xFF00u) << 16) | ((lb & 0xFF00u) << 8);
                    o[2 * c + 1] = ((sy >> 8) & 0xFF00u) | ((lb >> 16) & 0xFFu) | (sy & 0xFF000000u) | ((lb >> 8) & 0xFF0000u);
                }
                u32x4 a0;
                a0.x = o[0]; a0.y = o[1]; a0.z = o[2]; a0.w = o[3];
                *reinterpret_cast<u32x4 *>(out + i0) = a0;
            } else {
                for (uint32_t i = i0; i < gn; ++i) {                      // the ragged end of the bucket's payload
                    const uint32_t t = i / kVcSub, it = i % kVcSub;
                    out[i] = (uint16_t)((((s_sym[(it >> 2) * kSymPitch + t] >> (8u * (it & 3u))) & 0xFFu) << 8) | lo[i]);
                }
            }
        }
    } else {
        // any alignment: 8 loads in flight per thread
        for (uint32_t base = 0; base < gn; base += 8 * kThreads) {
            uint32_t lb[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) {
                const uint32_t i = base + u * kThreads + s;
                lb[u] = (i < gn) ? (uint32_t)lo[i] : 0u;
            }
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) {
                const uint32_t i = base + u * kThreads + s;
                if (i < gn) {
                    const uint32_t t = i / kVcSub, it = i % kVcSub;       // decoding thread, its it-th value
                    const uint32_t sym = (s_sym[(it >> 2) * kSymPitch + t] >> (8u * (it & 3u))) & 0xFFu;
                    out[i] = (uint16_t)((sym << 8) | lb[u]);
                }
            }
        }
    }
    if (bad) atomicOr(a.flags, kFlagBadIndex);
}

// ---------------------------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------------------------
__global__ void fill_u64_kernel(unsigned long long *p, uint64_t n, unsigned long long v) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// p[i*stride] = 0 for i < n
__global__ void zero_strided_kernel(uint32_t *p, uint64_t n, uint32_t stride) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i * stride] = 0u;
}

// two-stream read probe with extract's load shape; the XOR-reduction keeps the loads alive
template <int V, bool NT>
__global__ __launch_bounds__(kThreads) void stream_probe_kernel(const uint16_t *pa, const uint16_t *pb, uint64_t nvec,
                                                                 uint32_t *sink) {
    constexpr uint32_t TILE = (uint32_t)V * kUnit;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * TILE + (uint32_t)wave * (V * 512u) + (uint32_t)lane * 8u;
    u32x4 acc = {0, 0, 0, 0};
    u32x4 xa[V], xb[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const uint64_t e = base + j * 512;
        const bool ok = e / 8 < nvec;
        xa[j] = ok ? load16<NT>(as_global(pa) + e) : acc;
        xb[j] = ok ? load16<NT>(as_global(pb) + e) : acc;
    }
#pragma unroll
    for (int j = 0; j < V; ++j) acc ^= xa[j] ^ xb[j];
    uint32_t r = acc.x ^ acc.y ^ acc.z ^ acc.w;
    r = lane63(wave_inclusive_scan(r & 0xFFu));
    if (lane == 0 && wave == 0) sink[blockIdx.x] = r;
}

}  // namespace srs

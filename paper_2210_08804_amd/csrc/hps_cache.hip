// GPU embedding cache for MI355X (gfx950, wave64): kernels and the C ABI of include/hps_cache.h.
//
// Memory layout (all in HBM, owned by the cache):
//   K   int64  [S][W]      keys, one 64-byte line per set at W = 8; EMPTY = INT64_MIN
//   V   fp32   [S][W][d]   rows, 16-byte aligned, moved as opaque 128-bit chunks
//   sc  uint32 [S][2]      one 8-byte word per set: {seq, ctr}
//                            seq  sequence word: odd while a writer owns the set (lock + seqlock)
//                            ctr  victim counter: next way of the set = ctr mod W
//                          (together so that an insert gets both with its one 64-bit atomic and
//                          lets go of both with one store; every read is a 128-byte request)
//   T   uint32 [S][W]      access stamps, only for caches created with the LRU policy
//   epoch uint32 [16][64]  16 lines of {started, finished}: writer work-groups counted in and out
//
// Paper passages: data model Sec. 4.1; Query Alg. 2; Replace Alg. 3; Update Alg. 4; Dump and
// the asynchronous, batch-in calling convention Sec. 4.2.  The paper's per-slabset warp lock
// (Sec. 4.1) survives as the per-set sequence word, but only writers take it: query is
// read-only because the victim rule keeps no access stamps.
#include <hip/hip_runtime.h>

#include <atomic>
#include <climits>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <type_traits>
#include <unordered_map>

#include "hps_cache.h"
#include "hps_membench.h"
#include "hps_mix.h"
#include "hps_rows.h"

namespace {

constexpr int64_t  kEmpty      = INT64_MIN;
constexpr int      kBlock      = 256;          // threads per work-group: 4 waves of 64
constexpr int      kWave       = 64;
constexpr int      kWavesPerWg = kBlock / kWave;
constexpr uint32_t kMinKeysPerWave = 8;        // fewest keys that a query gives a worker wave
constexpr uint32_t kRing       = 1024;         // counter words per half of the pool (see counter_word)
constexpr uint64_t kMagic      = 0x4850534341434845ull;
// Every loop that waits for another kernel's writer to let go of a set gives up after this many
// rounds (a held set is released within microseconds; this many rounds take about a second) and
// raises HPS_FLAG_STUCK_SET in the cache's flag word, so that no wave can spin forever.
constexpr uint32_t kMaxRounds  = 1u << 16;
// Longest row (in fp32) that a query may read while writers run: a row is read whole (4 wave loads
// of 16 bytes per lane at this length) before it is validated and stored.
constexpr uint32_t kMaxCheckedDim = 1024;
// Writer epochs of a cache (see writer_enter): pairs of counters, one 256-byte line each.  Atomics
// on one line execute one after the other, 11 ns each; 4,096 work-groups with two atomics each
// cost a kernel of empty work-groups 94 us on one line, 7 us on 16 lines, 3 us on 64.  A reader
// looks at all of them with one wave load, one lane per line.
constexpr uint32_t kEpochs      = 16;
constexpr uint32_t kEpochStride = 64;          // uint32 words between pairs

typedef float f32x4 __attribute__((ext_vector_type(4)));   // one 16-byte chunk of a row

thread_local std::string g_err;

hps_status_t fail(hps_status_t code, const std::string &msg) {
    g_err = msg;
    return code;
}

#define HIP_TRY(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess)                                                           \
            return fail(e_ == hipErrorOutOfMemory ? HPS_ERR_OOM : HPS_ERR_DEVICE,        \
                        std::string(#expr) + ": " + hipGetErrorString(e_));              \
    } while (0)

// ------------------------------------------------------------------ device helpers

// Alg. 2 "slabsetHasher(q) mod |S|": upper hash half modulo the set count (mask when S is 2^k).
__device__ __forceinline__ uint32_t set_of(int64_t key, uint32_t S, uint32_t smask) {
    uint32_t h = (uint32_t)(mix64((uint64_t)key) >> 32);
    return smask ? (h & smask) : (h % S);
}

__device__ __forceinline__ bool is_reserved(int64_t key) { return key < kEmpty + 2; }

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }
// The wave's number in its work-group, as the scalar that it is.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)); }

__device__ __forceinline__ int64_t shfl64(int64_t v, int src) {
    int lo = __shfl((int)(uint32_t)(uint64_t)v, src, kWave);
    int hi = __shfl((int)(uint32_t)((uint64_t)v >> 32), src, kWave);
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Number of set bits of m below this lane.
__device__ __forceinline__ int rank_in(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Orders this wave's LDS traffic against itself (no instructions, compiler-only).
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename T> __device__ __forceinline__ T ld_agent(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ void st_agent(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Data that kernels overlapping on different streams share (keys, rows, counters of the cache):
// every such load/store is itself an agent-scope relaxed atomic of 4 or 8 bytes, or for rows an
// access of that scope of 16 (global_load / global_store with sc1: the access is performed at the memory side of the non-coherent per-XCD
// L2s, so it sees and is seen by every other agent-scope access of the device), and the order
// "sequence word, then data, then sequence word" is kept by waiting until the wave's outstanding
// vector memory operations have completed (s_waitcnt vmcnt(0)) between the steps: a wave's vector
// memory instruction counter reaches zero only when every earlier load has returned its data and
// every earlier store has been acknowledged by the level it was addressed to.
// The wait is the compiler's own s_waitcnt instruction (vmcnt(0), the other counters left alone:
// 0x0F70 in the gfx9 encoding), not inline assembly: the pass that places the waits in front of
// every use of a loaded register reads it and knows from there on that nothing is outstanding.
// Behind an assembly string it assumed that every row load might still be in flight and put a
// vmcnt(0) in front of each row store, so a wave had one store in flight at a time.
__device__ __forceinline__ void wait_vm0() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void shared_acquire() { wait_vm0(); }
__device__ __forceinline__ void shared_release() { wait_vm0(); }
__device__ __forceinline__ uint64_t shared_ld64(const uint64_t *p) { return ld_agent(p); }
__device__ __forceinline__ void shared_st64(uint64_t *p, uint64_t v) { st_agent(p, v); }
// A 16-byte chunk of a row with the same scope, in one instruction that the compiler counts among the outstanding
// operations like any other.  It is no atomic and need not be: a row is only stored by the one that holds its set, and what
// a reader loaded of it is used only if no writer was at work on it (copy_rows_quiet, copy_rows_checked).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 global_u32x4;
__device__ __forceinline__ u32x4 shared_ld128(const u32x4 *p) { return __builtin_amdgcn_global_load_b128((global_u32x4 *)p, "agent"); }
__device__ __forceinline__ void shared_st128(u32x4 *p, u32x4 v) { __builtin_amdgcn_global_store_b128((global_u32x4 *)p, v, "agent"); }

// Arguments that arrive in registers.  They go in vectors: the runtime takes a while for each argument of a launch (eight of
// them more 0.3 us of the host's time).
typedef uint64_t u64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <typename T> __device__ __forceinline__ T *global_at(uint64_t word) { return (T *)(__attribute__((address_space(1))) T *)word; }
inline uint64_t word_of(const void *p) { return (uint64_t)reinterpret_cast<uintptr_t>(p); }

struct alignas(64) Table {     // one cache as the kernels see it (one 64-byte line of the kernel arguments)
    int64_t  *K;
    float    *V;
    uint32_t *sc;              // [S][2]: {sequence word, victim counter} of a set
    uint32_t  S;
    uint32_t  smask;           // S - 1 when S is a power of two, else 0
    uint32_t *T;               // [S][W] access stamps, LRU policy only (else nullptr)
    uint32_t *gdev;            // the cache's global iteration count g of Alg. 2 (LRU policy): one device word
    uint32_t *flags;           // one word of HPS_FLAG_* bits raised by kernels
    uint32_t *epoch;           // kEpochs pairs {started, finished} of writer work-groups, kEpochStride words apart
};
static_assert(sizeof(Table) == 64, "one line of the kernel arguments per table");

__device__ __forceinline__ uint32_t *seq_of(uint32_t *sc, uint32_t set) { return sc + 2ull * set; }

// Writer epochs.  Every work-group of an insert or update kernel that has keys to handle counts
// itself in before it stores a key or a row and out after its last key and row have landed, on the pair
// (work-group's number) mod kEpochs.  A reader that finds started == finished in every pair, reads keys and rows,
// and then finds every pair unchanged knows that no writer was at work in between, so it need not
// look at the sequence words of its sets: a writer's count is at the memory side before its first
// store is issued (writer_entered) and its stores are there before it counts itself
// out, so a reader that saw any of those stores sees the pair changed or not yet even.
__device__ __forceinline__ uint32_t *epoch_of(uint32_t *epoch, uint32_t i) { return epoch + (i % kEpochs) * kEpochStride; }

// A wave's view of the pairs: lanes 0 .. kEpochs-1 hold {finished, started} of one pair each.
__device__ __forceinline__ uint64_t read_epochs(const uint32_t *epoch) {
    const uint32_t lane = (uint32_t)lane_id();
    return lane < kEpochs ? ld_agent(reinterpret_cast<const uint64_t *>(epoch + lane * kEpochStride)) : 0ull;
}

// A writer's work-group in LDS: waves still at work, and whether the work-group's count has arrived.  Together
// the two counts cost a call of a few keys 0.5 us and larger ones nothing (2^18 rows: 206.8 us with them,
// 206.4 without).
struct WriterGroup { uint32_t left, entered; };
// Called by all threads of the work-group at the start, with a barrier of the work-group to follow.  Wave 0's count is
// on its way when it returns.
__device__ __forceinline__ void writer_enter(uint32_t *pair, WriterGroup *w) {
    if (threadIdx.x == 0) {
        w->left = (uint32_t)kWavesPerWg;
        w->entered = 0u;
        __hip_atomic_fetch_add(pair, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
// Wave 0, right after a wait for its outstanding memory operations, which covers the count: tells the
// others.  Nothing that wave 0 does before depends on another wave.
__device__ __forceinline__ void writer_tell(WriterGroup *w, bool &told) {
    if (!told) __hip_atomic_store(&w->entered, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    told = true;
}
// Every wave, before it stores a key or a row.  The count's round trip runs beside the one in which
// the waves take their first sets (a wait for it at the start cost 0.8 us per call).
__device__ __forceinline__ void writer_entered(WriterGroup *w) {
    while (__hip_atomic_load(&w->entered, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0u)
        __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");                          // no store of the wave moves up
}
// Called by each wave of the work-group when its own keys and rows have landed.
__device__ __forceinline__ void writer_leave(uint32_t *pair, WriterGroup *w, bool told) {
    if (!told) wait_vm0();                                  // (wave 0 had no key to look at)
    writer_tell(w, told);
    if (lane_id() == 0 && __hip_atomic_fetch_sub(&w->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 1u)
        __hip_atomic_fetch_add(pair + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Division of a list of rows of C chunks into wave loads of 64 chunks.  Packed, so that a query's scalar
// arguments stay within two 64-byte lines.
struct ChunkStep {
    uint32_t C;                // chunks per row
    uint32_t packed;           // bits 0-16: inv, (lane * inv) >> 16 == lane / C for lane < 64; 17-23: 64 / C; 24-30: 64 mod C
    __host__ __device__ __forceinline__ uint32_t inv() const { return packed & 0x1FFFFu; }
    __host__ __device__ __forceinline__ uint32_t rows() const { return (packed >> 17) & 0x7Fu; }
    __host__ __device__ __forceinline__ uint32_t rest() const { return packed >> 24; }
};

// Row geometry shared by all copy loops: a row is C = d/4 chunks of 16 bytes; LPR lanes
// cooperate on one row (16 B per lane, contiguous, so a wave load covers 64/LPR whole rows).
struct RowGeom {
    uint32_t d;                // fp32 per row
    uint32_t C;                // 16-byte chunks per row
    uint32_t LPR;              // lanes per row: min(64, next power of two >= C)
    uint32_t lprShift;         // log2(LPR)
    uint32_t passes;           // ceil(C / LPR): > 1 only for rows longer than 1 KiB
    ChunkStep c16, c8;         // walks over the 16-byte and the 8-byte chunks (scoped accesses) of a list of rows
};

// Lane's place (row r of the list, chunk c of that row) in wave load after wave load of a list of
// rows whose chunks are numbered through, 64 of them to a wave load: every lane has a chunk to move
// whatever the row's length.
struct ChunkWalk {
    uint32_t r, c;
    __device__ __forceinline__ ChunkWalk(const ChunkStep &s, uint32_t lane) {
        r = (lane * s.inv()) >> 16;
        c = lane - r * s.C;
    }
    __device__ __forceinline__ void next(const ChunkStep &s) {
        r += s.rows();
        c += s.rest();
        if (c >= s.C) {
            c -= s.C;
            ++r;
        }
    }
    // Makes the walk opaque to the compiler, which would otherwise keep the places of a whole group of
    // wave loads in registers from the loads to the stores, or across groups, instead of three
    // additions each (64 registers for 16 wave loads).
    __device__ __forceinline__ void forget() { asm volatile("" : "+v"(r), "+v"(c)); }
};

// Copy `cnt` (> 0) rows listed in LDS: row srcRow[e] of `src` to row dstRow[e] of `dst`, for
// e < cnt.  A wave load/store moves 64 chunks of 16 bytes, of as many rows as that is.  The rows go in groups of U wave
// loads: a group's loads are ALL issued, one wait for them follows, then the group's stores go out back to back.  With
// U = 26 the 52 rows of a wave of the 106,496-key batch (two 512-byte rows per wave load) are one group, and every worker wave has
// its whole share of the batch in flight at once (stand-alone test bed: 18.3 us per launch; two alternating buffers of 2 wave
// loads 21.5, one buffer of 4 22.9, two groups of 15 20.3).  Non-temporal loads here cost 6 us (repeated keys live
// on L2 hits), non-temporal stores save 2 us (rows of `out` are written once and not read again here).
// arrived() is called once, when the last group's rows are in registers.
// kD = 128 fixes the row geometry at compile time (32 lanes per row, one pass, shifts instead of multiplications); behind a list of an
// odd number of rows its last entry stands once more (written by the caller), and no lane needs a condition.
// kD = 0 takes the geometry from g and walks over the chunks of the listed rows (ChunkWalk), four wave loads at a time as far as
// there are any; lanes beyond the list load entry 0 and store nothing.
template <int U, int kD = 0, typename SrcIdx, typename DstIdx, typename Arrived>
__device__ __forceinline__ void copy_rows(const RowGeom g, const float *__restrict__ src,
                                          float *__restrict__ dst, const SrcIdx *srcRow,
                                          const DstIdx *dstRow, uint32_t cnt, Arrived &&arrived) {
    static_assert(kD == 0 || kD == 128, "only the 128-word row is specialised");
    const uint32_t lane = (uint32_t)lane_id();
    if constexpr (kD == 128) {
        const uint32_t sub = lane >> 5;                          // two rows per wave load
        const uint32_t off = (lane & 31u) * 4;
        for (uint32_t e0 = 0; e0 < cnt; e0 += 2 * U) {
            f32x4 buf[U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (e0 + 2 * u < cnt)                                // uniform
                    buf[u] = *reinterpret_cast<const f32x4 *>(src + (uint64_t)srcRow[e0 + 2 * u + sub] * 128 + off);
            // One wait for the whole group, stated where the compiler can see it: it cannot count loads and stores under a
            // condition among the outstanding operations, and would make the later stores of a group wait for the earlier ones.
            __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0), other counters untouched
            if (e0 + 2 * U >= cnt) arrived();
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (e0 + 2 * u < cnt)
                    __builtin_nontemporal_store(buf[u], reinterpret_cast<f32x4 *>(dst + (uint64_t)dstRow[e0 + 2 * u + sub] * 128 + off));
        }
    } else {
        constexpr int Q = 4;                                     // wave loads per test for the end of the list
        static_assert(U % Q == 0, "whole blocks of wave loads");
        const uint32_t total = cnt * g.C;
        ChunkWalk in(g.c16, lane), out = in;
        out.forget();
        for (uint32_t q0 = 0; q0 < total; q0 += kWave * U) {
            f32x4 buf[U];
#pragma unroll
            for (int b = 0; b < U; b += Q) {
                if (q0 + b * kWave < total) {                    // uniform
#pragma unroll
                    for (int u = b; u < b + Q; ++u) {
                        const bool live = q0 + u * kWave + lane < total;
                        buf[u] = *reinterpret_cast<const f32x4 *>(src + (uint64_t)srcRow[live ? in.r : 0u] * g.d + (live ? in.c : 0u) * 4);
                        in.next(g.c16);
                    }
                }
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);                  // as above
            if (q0 + kWave * U >= total) arrived();
#pragma unroll
            for (int b = 0; b < U; b += Q) {
                if (q0 + b * kWave < total) {
#pragma unroll
                    for (int u = b; u < b + Q; ++u) {
                        if (q0 + u * kWave + lane < total)
                            __builtin_nontemporal_store(buf[u], reinterpret_cast<f32x4 *>(dst + (uint64_t)dstRow[out.r] * g.d + out.c * 4));
                        out.next(g.c16);
                    }
                }
            }
        }
    }
}

// copy_rows for a reader that found no writer at work when it read the epochs e1 (read_epochs).
// Rows are loaded 16 bytes per lane with shared_ld128, in groups of U wave loads, all of a group's
// loads in flight together; once they have completed the epochs are read again, and only if no
// writer has started meanwhile are the group's rows stored.  A row is always read whole inside one
// group (the longest, 4 KiB, takes 4 wave loads, which is why U >= 4 and why kMaxCheckedDim is
// 1024): a position whose key turns out to be gone when the rest is looked up again has had nothing
// written to its `out` row.  With kD = 128 two rows go in a wave load; behind a list of an odd number of rows its
// last entry stands once more (written by the caller), so that no lane needs a condition.
// Bound by memory, and before that by the loads' issue: half as many of them as with 8 bytes per lane take 106,496
// keys of 512 bytes from 19.7 to 18.0 us, 425,984 from 73 to 65, 851,968 of 128 bytes from 54 to 50, 20,000 of 4 KiB from 32.7 to 28.  Returns how many rows of the list are done; the caller goes through
// the others again with copy_rows_checked.
template <int U, int kD = 0, typename Tell>
__device__ __forceinline__ uint32_t copy_rows_quiet(const RowGeom g, const float *__restrict__ src,
                                                    float *__restrict__ dst, const uint64_t *srcRow,
                                                    const uint32_t *dstRow, uint32_t cnt,
                                                    uint64_t e1, const uint32_t *epoch, Tell &&tell) {
    static_assert((kD == 0 || kD == 128) && U >= 4 && (kD || U % 4 == 0), "a 512-byte row is half a wave load");
    constexpr int Q = kD ? 1 : 4;                                    // wave loads per test for the end of the list
    const uint32_t lane = (uint32_t)lane_id();
    const uint64_t d = kD ? (uint64_t)kD : (uint64_t)g.d;
    const uint32_t C = kD ? 32u : g.c16.C;
    const uint32_t span = kD ? (uint32_t)(2 * U) : (uint32_t)(U * kWave) / C;   // rows per group
    const ChunkWalk start(g.c16, lane);
    for (uint32_t e0 = 0; e0 < cnt; e0 += span) {
        const uint32_t rows = cnt - e0 < span ? cnt - e0 : span;
        const uint32_t total = rows * C;                             // chunks of the group
        u32x4 buf[U];
        ChunkWalk in = start, out = start;
        if (!kD) {
            in.forget();
            out.forget();
        }
#pragma unroll
        for (int b = 0; b < U; b += Q) {
            if ((uint32_t)b * kWave < total) {                       // uniform: there are chunks left
#pragma unroll
                for (int u = b; u < b + Q; ++u) {
                    const bool live = kD || u * kWave + lane < total;
                    const uint32_t r = kD ? 2 * u + (lane >> 5) : live ? in.r : 0u;
                    const uint32_t c = kD ? lane & 31u : live ? in.c : 0u;
                    buf[u] = shared_ld128(reinterpret_cast<const u32x4 *>(src + srcRow[e0 + r] * d) + c);
                    if (!kD) in.next(g.c16);
                }
            }
        }
        shared_acquire();                                            // row loads complete before the epochs are read again
        if (__ballot(read_epochs(epoch) != e1)) return e0;
        if (e0 + span >= cnt) tell();
#pragma unroll
        for (int b = 0; b < U; b += Q) {
            if ((uint32_t)b * kWave < total) {
#pragma unroll
                for (int u = b; u < b + Q; ++u) {
                    if (kD || u * kWave + lane < total)
                        __builtin_nontemporal_store(
                            buf[u], reinterpret_cast<u32x4 *>(dst + (uint64_t)dstRow[e0 + (kD ? 2 * u + (lane >> 5) : out.r)] * d) + (kD ? lane & 31u : out.c));
                    if (!kD) out.next(g.c16);
                }
            }
        }
    }
    if (cnt == 0) tell();
    return cnt;
}

// copy_rows for a reader that overlaps writers (seqlock read side).  Entry e also carries
// the set it came from and the value v1 of that set's sequence word read before the probe.
// Rows are loaded into registers (16 bytes per lane, shared_ld128), then the sequence words are
// read again once those loads have completed; a row is stored only if its word is unchanged,
// i.e. no writer touched the set while the row was being read.  Entries to redo are flagged in
// the LDS word pair `retry`.
// The wave's rows go in groups of U wave loads as in copy_rows_quiet; then ONE more wave load reads
// the sequence words again, lane l that of the group's row l, and a ballot of "changed" gives the
// rows to redo.  That is two dependent round trips per group, so the fewer groups the better (27.5 us
// per 106,496-key batch with groups of 16 rows, 21.6 us with one group per wave in the stand-alone
// test bed).
template <int U, int kD = 0>
__device__ __forceinline__ void copy_rows_checked(const RowGeom g, const float *__restrict__ src,
                                                  float *__restrict__ dst, const uint64_t *srcRow,
                                                  const uint32_t *dstRow, const uint32_t *setOf,
                                                  const uint32_t *v1Of, const uint32_t *sc,
                                                  uint32_t cnt, uint32_t *retry, uint32_t lane) {
    static_assert((kD == 0 || kD == 128) && U >= 4, "a 512-byte row is half a wave load");
    const uint64_t d = kD ? (uint64_t)kD : (uint64_t)g.d;
    const uint32_t C = kD ? 32u : g.c16.C;
    // rows per group: one lane per row re-reads its sequence word, so a group has at most 64 rows
    uint32_t span = kD ? (uint32_t)(2 * U) : (uint32_t)(U * kWave) / C;
    span = span < (uint32_t)kWave ? span : (uint32_t)kWave;
    const ChunkWalk start(g.c16, lane);
    for (uint32_t e0 = 0; e0 < cnt; e0 += span) {
        const uint32_t rows = cnt - e0 < span ? cnt - e0 : span;
        const uint32_t total = rows * C;                             // chunks of the group
        u32x4 buf[U];
        ChunkWalk in = start, out = start;
        if (!kD) {
            in.forget();
            out.forget();
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if ((uint32_t)u * kWave < total) {                       // uniform: there are chunks left
                const bool live = kD || u * kWave + lane < total;
                const uint32_t r = kD ? 2 * u + (lane >> 5) : live ? in.r : 0u;
                const uint32_t c = kD ? lane & 31u : live ? in.c : 0u;
                buf[u] = shared_ld128(reinterpret_cast<const u32x4 *>(src + srcRow[e0 + r] * d) + c);
                if (!kD) in.next(g.c16);
            }
        }
        shared_acquire();                                            // row loads complete before the re-read
        const bool mine = lane < rows + (kD ? rows & 1u : 0u);       // (the entry behind an odd list is a copy of its last)
        const uint32_t v2 = mine ? ld_agent(sc + 2ull * setOf[e0 + lane]) : 0u;
        const uint64_t bad = __ballot(mine && v2 != v1Of[e0 + lane]);   // bit r: row e0 + r was touched by a writer
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if ((uint32_t)u * kWave < total) {
                const uint32_t r = kD ? 2 * u + (lane >> 5) : out.r;
                const uint32_t c = kD ? lane & 31u : out.c;
                if ((kD || u * kWave + lane < total) && !((bad >> r) & 1ull))
                    __builtin_nontemporal_store(buf[u], reinterpret_cast<u32x4 *>(dst + (uint64_t)dstRow[e0 + r] * d) + c);
                if (!kD) out.next(g.c16);
            }
        }
        if (bad && lane == 0) {                                      // e0 + rows <= cnt <= 64
            const uint64_t m = bad << e0;
            __hip_atomic_fetch_or(retry + 0, (uint32_t)m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_fetch_or(retry + 1, (uint32_t)(m >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
}

// Writer side: the rows listed in LDS go from the caller's batch into the cache with agent-scope stores, so that
// overlapping readers observe them without cache flushes.  start() requests the
// first two groups of U wave loads; finish() stores them and moves what is left, each group's loads
// issued before the stores of the group ahead of it, so that a write-through store's long
// acknowledgement never sits between a wave and its next loads.  The two halves are apart because
// which rows are read may be known long before it is known which of them are to be stored.
// Rows of up to 1 KiB (kLong false) take LPR lanes of 16 bytes each, a whole number of them per wave load; longer
// ones go, 8 bytes per lane, through the walk over the chunks of the list, so that no wave load is partly idle and
// the parts of a row are in flight together (30,000 rows of 1,280 bytes inserted, updated and queried:
// 93.6 us when each 512-byte part of the rows was a pass of its own, 71 us with the walk).  For shorter
// rows the walk's arithmetic costs more than it saves (400-byte rows 41.7 against 38.7 us, 30,000 rows of 768 / 1,024 bytes inserted,
// updated and queried 55.9 / 61.9 against 54.4 / 60.4).  A walk in pieces of 16 bytes has not been measured.
// Bound by memory and by the chain around the copy.  16 bytes per lane instead of 8, half as many loads and stores: 2^18 rows of 512
// bytes inserted, updated and queried 206.3 -> 197.2 us, 200,000 rows of 400 bytes 172 -> 159, 1 GiB of rows refreshed 446 -> 438.
// (Twice as many wave loads in flight, U = 8: 200.4 and 441 us.  Plain write-back stores 198.1 and 455, non-temporal ones 213 and 424, and
// neither could be seen by a reader in time.  Groups of 16 or 32 wave loads all in flight before the first store, which is
// what the query's copy does, cost the writers occupancy and time, measured with 8 bytes per lane: insert 102 us against 83 us per 2^18 rows, update 118
// against 81 us.)
constexpr uint64_t kSkipRow = ~0ull;             // dstRow of an entry that finish() is not to store

// What a lane moves of a row at a time: 8 bytes of a long row, 16 of a shorter one.
template <bool kLong>
struct RowPiece {
    typedef uint64_t type;
    static __device__ __forceinline__ type load(const float *row, uint32_t c) { return __builtin_nontemporal_load(reinterpret_cast<const uint64_t *>(row) + c); }
    static __device__ __forceinline__ void store(float *row, uint32_t c, type v) { shared_st64(reinterpret_cast<uint64_t *>(row) + c, v); }
    static __device__ __forceinline__ const ChunkStep &step(const RowGeom &g) { return g.c8; }
};
template <>
struct RowPiece<false> {
    typedef u32x4 type;
    static __device__ __forceinline__ type load(const float *row, uint32_t c) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(row) + c); }
    static __device__ __forceinline__ void store(float *row, uint32_t c, type v) { shared_st128(reinterpret_cast<u32x4 *>(row) + c, v); }
    static __device__ __forceinline__ const ChunkStep &step(const RowGeom &g) { return g.c16; }
};

template <int U, bool kLong>
struct RowMover {
    typedef RowPiece<kLong> P;
    typedef typename P::type Chunk;
    const RowGeom &g;
    const float *const src;
    float *const dst;
    const uint32_t *const srcRow;
    const uint64_t *const dstRow;
    uint32_t cnt;
    ChunkWalk in, out;
    Chunk bufA[U], bufB[U];

    __device__ __forceinline__ RowMover(const RowGeom &g_, const float *src_, float *dst_, const uint32_t *srcRow_, const uint64_t *dstRow_)
        : g(g_), src(src_), dst(dst_), srcRow(srcRow_), dstRow(dstRow_), cnt(0), in(P::step(g_), (uint32_t)lane_id()), out(in) {}

    // Wave load k of the list: does it hold rows at all (uniform), does this lane have one, which row, which chunk of it.
    __device__ __forceinline__ bool any(uint32_t k) const {
        return kLong ? (uint64_t)k * kWave < (uint64_t)cnt * P::step(g).C : (k << (6u - g.lprShift)) < cnt;
    }
    __device__ __forceinline__ bool place(uint32_t k, ChunkWalk &w, uint32_t &r, uint32_t &c) const {
        const uint32_t lane = (uint32_t)lane_id();
        bool live;
        if (kLong) {
            live = w.r < cnt;
            r = live ? w.r : 0u;
            c = live ? w.c : 0u;
            w.next(P::step(g));
        } else {
            const uint32_t e = (k << (6u - g.lprShift)) + (lane >> g.lprShift);
            live = e < cnt;
            r = live ? e : 0u;
            c = lane & (g.LPR - 1u);
            c = c < P::step(g).C ? c : 0u;
        }
        return live;
    }
    __device__ __forceinline__ void load(uint32_t k, Chunk (&buf)[U]) {       // lanes past the list read entry 0
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t r, c;
            (void)place(k + u, in, r, c);
            buf[u] = P::load(src + (uint64_t)srcRow[r] * g.d, c);
        }
    }
    // A whole group of rows that are all to be stored goes out in one piece.  Otherwise the wait comes first: the
    // compiler cannot count predicated stores among the outstanding operations.
    __device__ __forceinline__ void put(uint32_t k, const Chunk (&buf)[U], bool all) {
        if (all && any(k + U - 1)) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                uint32_t r, c;
                (void)place(k + u, out, r, c);
                P::store(dst + dstRow[r] * g.d, c, buf[u]);
            }
        } else {
            wait_vm0();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!any(k + u)) break;
                uint32_t r, c;
                const bool live = place(k + u, out, r, c);
                const uint64_t row = dstRow[r];
                if (live && row != kSkipRow) P::store(dst + row * g.d, c, buf[u]);
            }
        }
    }
    __device__ __forceinline__ void start(uint32_t cnt_) {
        cnt = cnt_;
        if (kLong) {
            in = out = ChunkWalk(P::step(g), (uint32_t)lane_id());
            out.forget();
        }
        load(0, bufA);
        if (any(U)) load(U, bufB);
    }
    __device__ __forceinline__ void finish(bool all) {
        for (uint32_t k = 0;;) {
            put(k, bufA, all);
            if (any(k + 2 * U)) load(k + 2 * U, bufA);
            if (!any(k += U)) return;
            put(k, bufB, all);
            if (any(k + 2 * U)) load(k + 2 * U, bufB);
            if (!any(k += U)) return;
        }
    }
};

// The same in one go, for rows that are all stored.
template <int U, bool kLong>
__device__ __forceinline__ void copy_rows_shared(const RowGeom &g, const float *__restrict__ src,
                                                 float *dst, const uint32_t *srcRow,
                                                 const uint64_t *dstRow, uint32_t cnt) {
    typedef RowPiece<kLong> P;
    typedef typename P::type Chunk;
    const uint32_t lane = (uint32_t)lane_id();
    const uint32_t rpi = (uint32_t)kWave >> g.lprShift;
    const uint32_t sub = lane >> g.lprShift;
    uint32_t cl = lane & (g.LPR - 1);
    cl = cl < P::step(g).C ? cl : 0u;
    typedef typename std::conditional<kLong, uint64_t, uint32_t>::type Count;   // 16 rows of 2 GiB have 2^32 chunks
    const Count step = kLong ? (Count)(kWave * U) : (Count)(rpi * U);
    const Count total = kLong ? (Count)cnt * P::step(g).C : (Count)cnt;     // chunks, or rows
    Chunk bufA[U], bufB[U];
    uint32_t entA[U], entB[U], offA[kLong ? U : 1], offB[kLong ? U : 1];
    ChunkWalk in(P::step(g), lane);
    auto load = [&](Count q0, Chunk (&buf)[U], uint32_t (&ent)[U], uint32_t *off) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kLong) {
                const bool live = in.r < cnt;
                ent[u] = live ? in.r : 0u;
                off[u] = live ? in.c : 0u;
                in.next(P::step(g));
            } else {
                const uint32_t e = (uint32_t)q0 + u * rpi + sub;
                ent[u] = e < cnt ? e : 0u;
            }
            buf[u] = P::load(src + (uint64_t)srcRow[ent[u]] * g.d, kLong ? off[u] : cl);
        }
    };
    auto store = [&](const Chunk (&buf)[U], const uint32_t (&ent)[U], const uint32_t *off) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            P::store(dst + dstRow[ent[u]] * g.d, kLong ? off[u] : cl, buf[u]);
    };
    load(0, bufA, entA, offA);
    for (Count q0 = 0;; q0 += 2 * step) {
        load(q0 + step, bufB, entB, offB);
        store(bufA, entA, offA);
        if (q0 + step >= total) break;
        load(q0 + 2 * step, bufA, entA, offA);
        store(bufB, entB, offB);
        if (q0 + 2 * step >= total) break;
    }
}

// Set probe for the first KPW lanes' keys of a wave (Alg. 2 "warpReadOutSlab" + match): W lanes
// read the W slot keys of one set (contiguous 8*W bytes), so one wave load covers 64/W sets; a
// ballot over the equality test gives every key its way.  Returns the way or -1.  between() runs after
// the loads of the (last) round have been issued: it may issue further loads behind them.  Only the first `lanes`
// lanes have keys; with sets of 32 ways and more a wave load covers two keys or one, and those of the other lanes are left out
// (40,000 keys of 512 bytes in 64-way sets, 24 keys per wave, checked: 16.1 us with them, all on the line of set 0, 11.3 without).
// A lane that wants nothing seeks a value that no slot holds: its key travels alone, one shuffle in four less than with its `want` beside it.
template <int W, int KPW, bool kShared = false, typename Between>
__device__ __forceinline__ int probe_wave(const int64_t *__restrict__ K, int64_t key,
                                          uint32_t set, bool want, Between &&between, uint32_t lanes = KPW, int lane = lane_id()) {
    constexpr int G = kWave / W;                       // keys per wave load
    constexpr int R = (KPW + G - 1) / G;               // wave loads needed for KPW keys
    constexpr int RC = R > 32 ? 32 : R;                // wave loads in flight together (64 for W = 64 would not fit the registers)
    const int slot = lane & (W - 1);
    const int sub  = lane / W;
    int way = -1;
    const int64_t sought = want ? key : kEmpty + 1;
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += RC) {
        int64_t sk[RC];
        constexpr int RB = W >= 32 && RC >= 8 ? 8 : RC;              // wave loads per test for lanes that have keys
#pragma unroll
        for (int b = 0; b < RC; b += RB) {
            if (RB < RC && (uint32_t)((r0 + b) * G) >= lanes) continue;   // uniform
#pragma unroll
            for (int r = b; r < b + RB; ++r) {
                const int j = (r0 + r) * G + sub;
                const uint32_t sj = (uint32_t)__shfl((int)set, j, kWave);   // 0 for lanes without a key: a valid set
                const int64_t *p = K + (uint64_t)sj * W + slot;
                sk[r] = kShared ? (int64_t)shared_ld64(reinterpret_cast<const uint64_t *>(p)) : *p;
            }
        }
        if (r0 + RC >= R) between();
#pragma unroll
        for (int b = 0; b < RC; b += RB) {
            if (RB < RC && (uint32_t)((r0 + b) * G) >= lanes) continue;
#pragma unroll
            for (int r = b; r < b + RB; ++r) {
                const int j = (r0 + r) * G + sub;
                const int64_t kj = shfl64(sought, j);
                const uint64_t m = __ballot(sk[r] == kj);
                if (lane / G == r0 + r) {
                    const uint64_t field = (W == 64) ? m : ((m >> ((lane % G) * W)) & ((1ull << (W & 63)) - 1));
                    if (field) way = __builtin_ctzll(field);
                }
            }
        }
    }
    return want ? way : -1;
}
template <int W, int KPW, bool kShared = false>
__device__ __forceinline__ int probe_wave(const int64_t *__restrict__ K, int64_t key, uint32_t set, bool want, uint32_t lanes = KPW) {
    return probe_wave<W, KPW, kShared>(K, key, set, want, [] {}, lanes);
}

// probe_wave for an insert with the LRU policy: the stamps of the sets travel with their keys, and `victim` becomes the way that
// a new key takes (Alg. 3): the lowest empty one, else that of the oldest stamp, the lowest of them.  W lanes work on a set, so
// the choice costs no round trip; a lane that asked for its W keys and stamps by itself, behind the search, waited for most of them
// one by one (8 ways, 512-byte rows, new keys: 262,144 over 2^20 sets 113.9 -> 82.4 us, 70,000 over 2^16 48.9 -> 38.8, 8,192 over 2^11 41.5 -> 28.7).
template <int W, int KPW, int kMost, typename Between>
__device__ __forceinline__ int probe_lru_wave(const int64_t *K, const uint32_t *T, int64_t key, uint32_t set, bool want, uint32_t g_now,
                                              int &victim, int lane, Between &&between) {
    constexpr int G = kWave / W;                       // keys per wave load
    constexpr int R = (KPW + G - 1) / G;               // wave loads needed for KPW keys
    constexpr int RC = R > kMost ? kMost : R;          // wave loads in flight together
    const int slot = lane & (W - 1);
    const int sub  = lane / W;
    int way = -1;
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += RC) {
        int64_t  sk[RC];
        uint32_t stamp[RC];
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            const uint32_t sj = (uint32_t)__shfl((int)set, (r0 + r) * G + sub, kWave);   // 0 for lanes without a key: a valid set
            const uint64_t at = (uint64_t)sj * W + slot;
            sk[r] = (int64_t)shared_ld64(reinterpret_cast<const uint64_t *>(K + at));
            stamp[r] = ld_agent(T + at);
        }
        if (r0 + RC >= R) between();
#pragma unroll
        for (int r = 0; r < RC; ++r) {
            const int j = (r0 + r) * G + sub;
            const int64_t kj = shfl64(key, j);
            const int wj = __shfl((int)want, j, kWave);
            const uint32_t age = g_now - stamp[r];
            uint32_t oldest = age;
#pragma unroll
            for (int o = 1; o < W; o <<= 1) {
                const uint32_t other = (uint32_t)__shfl_xor((int)oldest, o, kWave);
                oldest = other > oldest ? other : oldest;
            }
            const uint64_t same = __ballot(wj && sk[r] == kj), empty = __ballot(sk[r] == kEmpty), old = __ballot(age == oldest);
            if (lane / G == r0 + r) {
                const int at = W == 64 ? 0 : (lane % G) * W;
                constexpr uint64_t all = W == 64 ? ~0ull : (1ull << (W & 63)) - 1;
                const uint64_t f = (same >> at) & all, e = (empty >> at) & all;
                if (f) way = __builtin_ctzll(f);
                victim = __builtin_ctzll(e ? e : (old >> at) & all);     // (some lane has the largest age)
            }
        }
    }
    return way;
}

// ------------------------------------------------------------------ query

// The scalars come first, in two 64-byte lines, then one line per table: a kernel's first reads of
// its arguments miss in the scalar cache line by line.  (What query_kernel needs for its first loads it is given in registers.)
struct QueryArgs {
    const int64_t *keys;        // [T][B]
    float         *out;         // [T][B][d]
    uint32_t      *miss_idx;
    int64_t       *miss_keys;
    uint32_t      *n_miss;
    uint64_t      *slot;        // the stream's counter word: low 32 bits = misses so far, high 32 = tiles done
    const uint32_t *n_dev;      // optional: the real batch length (<= B) is read on the device (one table only)
    uint32_t       B;           // keys per table
    uint32_t       kpw;         // keys per worker wave (<= 64): lanes kpw..63 of a worker wave stay idle
    uint32_t       tiles_per_table;
    uint32_t       n_tiles;     // T * tiles_per_table (>= 1 even when B == 0)
    uint32_t       n_tables;    // T (<= HPS_MAX_TABLES <= 64: one helper lane per table finishes the call)
    uint32_t       deal;        // keys that a wave takes at a time of a batch whose length is read on the device (a power of two), 0: its kpw
    RowGeom        g;
    Table          tab[HPS_MAX_TABLES];
};
static_assert(offsetof(QueryArgs, tab) == 128, "two lines of scalars");
// Where query_kernel's QueryArgs stand in its argument block: behind 14 words of its own, at the next multiple of their alignment.
constexpr uint32_t kQueryArgsAt = 64;
static_assert(alignof(QueryArgs) == 64, "kQueryArgsAt");
typedef const __attribute__((address_space(4))) QueryArgs *QueryArgsIn;
constexpr uint32_t kGridX = 1u << 20;          // work-groups in a row of a query's grid

// Kernel arguments are read with scalar loads where they are first used, each followed by its own
// wait; spread over several cache lines and basic blocks that put three to five dependent
// scalar-cache misses in front of a wave's first key load (0.7 us of a 19 us query launch).  The
// kernels therefore name everything a tile needs in ONE empty asm statement: all the loads are
// issued together ahead of it and waited for once.
#define HPS_ARGS_NOW(...) asm volatile("" ::__VA_ARGS__)

// What the tile that finds every other tile of its call finished does (helper wave, all lanes):
// publish the miss count, clear the call's counter word for the next call on the stream, and
// advance the iteration count g of every LRU table of the call (Alg. 2 has thread 0 do the
// atomic add; every tile has read g by then, because a tile reads it before it adds its count).
// gdev: lane t's word of table t, nullptr for a table without stamps.
__device__ __forceinline__ void finish_call(uint32_t *n_miss, uint64_t *slot, uint32_t *gdev, uint32_t misses, int lane) {
    if (lane == 0) {
        *n_miss = misses;
        __hip_atomic_store(slot, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (gdev) __hip_atomic_fetch_add(gdev, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Query (Alg. 2).  A work-group is WPB worker waves plus one helper wave and handles one tile of
// WPB*kpw positions; the first kpw lanes of each worker wave own one key each.
//   workers  load key, hash, probe the set (probe_wave); misses are compacted per wave into LDS
//            (ballot + mbcnt prefix), hits into the wave's <source slot, destination position>
//            list; the wave then copies its rows without waiting for the others.
//   helper   once every worker wave has its rows (an LDS counter) it adds the tile's miss count to the call's counter
//            word with one 64-bit atomic (low half: misses so far, high half: tiles done), then
//            writes the tile's miss entries from LDS to the global list.  The tile that finds
//            every other tile done publishes *n_miss and clears the word for the next call.
// The helper exists so that no worker has the atomic's round trip in front of its row loads
// (vector memory results return in issue order).  It is told between a wave's loads and its stores: the tiles' atomics go to one
// address, one after the other, and hold up what else goes to that channel, which a wave waits for while it reads rows and
// nobody does while they are written (told as soon as the misses were known: 39,999 keys of 1,280 bytes plain 18.6 us, this way 15.7; 106,496 of
// 512 bytes 17.3, 16.3; 26 tables 214, 208).  Where a wave has little to read, or few tiles meet, nothing waits for the atomics but the end of the call: plain waves of up to
// 8 KiB of rows (12 KiB in up to 192 tiles of 512-byte rows) tell at once.  (Behind the loads / at once, us: 2 tables x 858 keys of 128 bytes 4.1 / 3.8, 4,907 keys of 512 bytes 4.6 / 4.2,
// 118,205 keys of 128 bytes 8.3 / 7.3; but 64 keys of 256 bytes to a wave, 30,926 keys of 1 KiB 1.17 times as long.  Rows that come from 8 GiB of memory, 512 bytes: 6,656 keys, 17 to a wave, 6.0 / 5.5,
// 9,620, 24 to a wave, 6.3 / 6.3, 13,312, 32 to a wave, 6.8 / 7.2, 26,624 7.8 / 8.7, 39,936 8.8 / 10.4.)
// One tile to a work-group, and no loop over tiles around it: what a loop keeps in registers from one tile to the next took up to 100 more of
// them, and as long before the first load (registers plain / checked, 512-byte rows in groups of 32: 221 / 237 with the loop, 138 / 151 without,
// 128-byte rows checked 103, 62).  The first 14 words of the arguments arrive in registers (-amdgpu-kernarg-preload-count), so that a
// wave's keys are requested ahead of the scalar loads for the rest, on which they waited before.  Both together with the above, us: 26,624 keys under LRU
// 10.6 -> 9.2, 106,496 keys plain 17.9 -> 17.0 and checked 18.0 -> 16.7, 851,968 of 128 bytes checked 49.8 -> 44.5, 47,000 distinct keys
// through a length on the device 12.6 -> 11.
//
// kCoherent = true is the variant for queries that may overlap insert/update kernels on other
// streams: each worker reads its sets' sequence words before probing, skips sets a writer holds
// (odd word), copies rows with copy_rows_checked and repeats for the keys whose set changed under
// it.  A miss needs no check (an 8-byte key is read whole, and a key that stays cached is never
// absent from its slot), so only hits are validated.
// kFull = true is launched for calls that name an LRU table or take their length from the device
// (n_dev): only those kernels read g, stamp their hits and read *n_dev.  (As never-taken branches
// in every kernel the three cost 0.4 us of a 19 us launch.)
template <int W, int KPW, int U, int WPB, bool kCoherent, int kD = 0, bool kFull = false>
__global__ void __launch_bounds__((WPB + 1) * kWave)
query_kernel(const u64x4 pointers, const u32x4 sizes, const u32x2 sets, const QueryArgs) {
    const int64_t *__restrict__ const keys = global_at<const int64_t>(pointers.x);
    const int64_t *const K0 = global_at<const int64_t>(pointers.y);
    const uint32_t *const epoch0 = global_at<const uint32_t>(pointers.z);
    const uint32_t *const n_dev = global_at<const uint32_t>(pointers.w);
    const uint32_t batch = sizes.x, kpw = kFull ? sizes.y & 0xFFFFu : sizes.y, deal = kFull ? sizes.y >> 16 : 0u, tiles_per_table = sizes.z, n_tiles = sizes.w, S0 = sets.x, smask0 = sets.y;
    __shared__ uint64_t s_src[WPB][KPW];                // (an odd number of rows is less than KPW: room for its copied last entry)
    __shared__ uint32_t s_dst[WPB][KPW];
    __shared__ int64_t  s_mkey[WPB][KPW];
    __shared__ uint32_t s_mpos[WPB][KPW];
    __shared__ uint32_t s_wcnt[WPB];
    __shared__ uint32_t s_ready;                   // worker waves that have listed their misses
    __shared__ uint32_t s_set[kCoherent ? WPB : 1][kCoherent ? KPW : 1];
    __shared__ uint32_t s_v1[kCoherent ? WPB : 1][kCoherent ? KPW : 1];
    __shared__ uint32_t s_retry[kCoherent ? WPB : 1][2];

    const int lane = lane_id();
    const int wave = wave_id();
    const uint32_t tile = blockIdx.y * kGridX + blockIdx.x;
    if (tile >= n_tiles) return;                       // the grid's last row need not be full
    const bool one = tiles_per_table == n_tiles;       // a call on one table
    uint32_t t = 0u, lt = tile;
    if (!one) {
        t  = tile / tiles_per_table;
        lt = tile - t * tiles_per_table;
    }
    QueryArgsIn in = (QueryArgsIn)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + kQueryArgsAt);
    if (threadIdx.x == 0) s_ready = 0u;
    // A length that is read on the device: its keys are dealt to all the waves launched for the longest one, `deal` neighbours (deal_of) at a
    // time, so that a wave's keys can be requested beside it (50,000 of 106,496 keys: all in the first half of the waves 20.0 us, spread 14.6).
    // At most kpw, rounded up to whole deals, fall to a wave.  Tiles to which none fall leave, and are not counted (4,000 of 200,000 keys plain 9.5 -> 5.2,
    // 3,000 of 300,000 plain 14.0 -> 5.6, in the default mode 13.5 -> 5.9).
    const bool dealt = kFull && deal;
    const uint32_t shift = dealt ? 31u - (uint32_t)__builtin_clz(deal) : 0u;
    auto tiles_of = [&](uint32_t nd) {
        const uint32_t deals = (nd >> shift) + ((nd & (deal - 1)) != 0), m = deals / WPB + (deals % WPB != 0);
        return !dealt ? n_tiles : m == 0 ? 1u : m < n_tiles ? m : n_tiles;
    };

    if (wave >= WPB) {
        // ---- helper
        uint32_t counted = n_tiles;
        if (kFull && n_dev) {
            const uint32_t nd = *n_dev;
            counted = tiles_of(nd < batch ? nd : batch);
            if (tile >= counted) return;
        }
        __syncthreads();
        uint32_t *const miss_idx = in->miss_idx, *const n_miss = in->n_miss;
        int64_t *const miss_keys = in->miss_keys;
        uint64_t *const slot = in->slot;
        HPS_ARGS_NOW("s"(miss_idx), "s"(miss_keys), "s"(slot), "s"(n_miss));
        // (looked up now: behind the last tile's atomic the call would wait for it)
        uint32_t *const gdev = kFull && (uint32_t)lane < in->n_tables && in->tab[lane].T ? in->tab[lane].gdev : nullptr;
        // every worker wave of the work-group reaches its increment (none leaves early), so this ends
        while (__hip_atomic_load(&s_ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < (uint32_t)WPB)
            __builtin_amdgcn_s_sleep(kCoherent ? 1 : 2);
        uint32_t total = 0;
#pragma unroll
        for (int w = 0; w < WPB; ++w) total += s_wcnt[w];
        uint64_t old = 0;
        if (lane == 0)
            old = __hip_atomic_fetch_add(slot, (1ull << 32) | (uint64_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        old = (uint64_t)shfl64((int64_t)old, 0);
        uint32_t o = (uint32_t)old;
#pragma unroll
        for (int w = 0; w < WPB; ++w) {
            const uint32_t c = s_wcnt[w];
            for (uint32_t j = (uint32_t)lane; j < c; j += kWave) {
                miss_idx[o + j]  = s_mpos[w][j];
                miss_keys[o + j] = s_mkey[w][j];
            }
            o += c;
        }
        if ((uint32_t)(old >> 32) + 1u == counted)     // every tile has added its count (and read g)
            finish_call(n_miss, slot, gdev, (uint32_t)old + total, lane);
        return;
    }

    // ---- worker
    const int64_t *K = K0;
    const uint32_t *epoch = epoch0;
    uint32_t S = S0, smask = smask0;
    if (!one) {
        K = in->tab[t].K;
        epoch = in->tab[t].epoch;
        S = in->tab[t].S;
        smask = in->tab[t].smask;
        if (kCoherent) HPS_ARGS_NOW("s"(K), "s"(epoch), "s"(S), "s"(smask));
        else           HPS_ARGS_NOW("s"(K), "s"(S), "s"(smask));
    }
    uint32_t b = (lt * WPB + wave) * kpw + lane;
    if (dealt) b = ((((uint32_t)lane >> shift) * (n_tiles * WPB) + lt * WPB + wave) << shift) + ((uint32_t)lane & (deal - 1));
    bool          live = (lane < (int)kpw || dealt) && b < batch;
    const uint32_t pos = t * batch + b;                // position in keys/out (< 2^32 checked on host)

    const int64_t  key = live ? keys[pos] : kEmpty;
    const uint64_t e1  = kCoherent ? read_epochs(epoch) : 0ull;
    if (kFull && n_dev) {
        const uint32_t nd = *n_dev;
        if (tile >= tiles_of(nd < batch ? nd : batch)) return;
        live = live && b < nd;
    }
    // Lanes up to the last that has a key: a length on the device leaves a wave some of those that a full batch would fill (64 ways, rows
    // of 512 bytes, 24,000 of 118,587 keys in the default mode 12.6 -> 9.5 without them).
    const uint32_t lanes = dealt ? kWave - (uint32_t)__builtin_clzll(__ballot(live) | 1ull) : kpw;
    __syncthreads();                                   // s_ready is zero
    __builtin_amdgcn_sched_barrier(0);                 // (nobody waits here for keys)
    // All that is needed from here on, while the keys travel.
    asm volatile("" : "+s"(in));
    float *const V = in->tab[t].V, *const out = in->out;
    uint32_t *const T = in->tab[t].T, *const sc = in->tab[t].sc;
    const RowGeom g = {in->g.d, in->g.C, in->g.LPR, in->g.lprShift, in->g.passes, {in->g.c16.C, in->g.c16.packed}, {in->g.c8.C, in->g.c8.packed}};
    HPS_ARGS_NOW("s"(V), "s"(out), "s"(T), "s"(sc), "s"(g.d), "s"(g.c16.C), "s"(g.c16.packed));
    // Alg. 2 "g <- g + 1": every tile of the call stamps with the count the call will leave
    // behind; the tile that finishes the call stores it (finish_call).
    const uint32_t g_call = kFull && T ? *in->tab[t].gdev + 1u : 0u;
    const bool     want = live && !is_reserved(key);
    const uint32_t set = want ? set_of(key, S, smask) : 0u;

    // A wave's misses go to LDS, the helper is told.
    uint32_t n_missed = 0;
    auto list_misses = [&](bool missed) {
        const uint64_t m = __ballot(missed);
        if (missed) {
            const uint32_t r = n_missed + (uint32_t)rank_in(m);
            s_mpos[wave][r] = pos;
            s_mkey[wave][r] = key;
        }
        n_missed += (uint32_t)__popcll(m);
    };
    auto tell = [&] {
        if (lane == 0) {
            s_wcnt[wave] = n_missed;
            __hip_atomic_fetch_add(&s_ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    // Alg. 2: refresh the counter.  A plain store: the XCD's write-back L2 merges the many stores
    // a hot key draws (an agent-scope store per hit serialises them at the memory side and
    // triples the kernel time); they reach memory at the latest when the kernel ends.
    auto stamp = [&](bool hit, int way) {
        if (kFull && T && hit) T[(uint64_t)set * W + (uint32_t)way] = g_call;
    };

    if constexpr (!kCoherent) {
        const int  way = probe_wave<W, KPW, false>(K, key, set, want, lanes);
        const bool hit = way >= 0;
        list_misses(live && !hit);
        const uint64_t hitmask = __ballot(hit);
        const uint32_t nh      = (uint32_t)__popcll(hitmask);
        if (hit) {
            const int r = rank_in(hitmask);
            s_src[wave][r] = (uint64_t)set * W + (uint32_t)way;
            s_dst[wave][r] = pos;
            if (kD && (nh & 1u) && r + 1 == (int)nh) {
                s_src[wave][nh] = (uint64_t)set * W + (uint32_t)way;
                s_dst[wave][nh] = pos;
            }
        }
        stamp(hit, way);
        wave_lds_fence();
        const bool early = n_tiles <= 192 ? U <= 8 || (kD && U <= 16 && kpw <= 24) : U <= 8 && W <= 16;
        if (early || !nh) tell();
        if (nh) copy_rows<U, kD>(g, V, out, &s_src[wave][0], &s_dst[wave][0], nh, [&] { if (!early) tell(); });
    } else {
        bool pending = want;
        list_misses(live && !want);
        // No writer at work.  (A wave without keys, of which a length on the device can leave most, has nothing to
        // look for: 3,000 of 300,000 keys 14.5 us if it does, 12.9 if not, while work-groups without keys stayed.)
        if (__ballot(want) && !__ballot((uint32_t)e1 != (uint32_t)(e1 >> 32))) {
            shared_acquire();                          // the epochs are read before any key or row
            const int way = probe_wave<W, KPW, true>(K, key, set, want, lanes);
            const uint64_t fmask = __ballot(way >= 0);
            const int r = rank_in(fmask);
            const uint32_t nf = (uint32_t)__popcll(fmask);
            if (way >= 0) {
                s_src[wave][r] = (uint64_t)set * W + (uint32_t)way;
                s_dst[wave][r] = pos;
                if (kD && (nf & 1u) && r + 1 == (int)nf) {
                    s_src[wave][nf] = (uint64_t)set * W + (uint32_t)way;
                    s_dst[wave][nf] = pos;
                }
            }
            list_misses(want && way < 0);              // a miss is final
            wave_lds_fence();
            const uint32_t done = copy_rows_quiet<U, kD>(g, V, out, &s_src[wave][0], &s_dst[wave][0], nf, e1, epoch, tell);
            const bool hit = way >= 0 && (uint32_t)r < done;
            stamp(hit, way);
            pending = way >= 0 && !hit;
            if (!__ballot(pending)) return;            // the helper has been told
            wave_lds_fence();
        }
        uint32_t rounds = 0;
        while (__ballot(pending)) {
            if (++rounds > kMaxRounds) {               // a set never came free: report a miss
                if (pending) __hip_atomic_fetch_or(in->tab[t].flags, (uint32_t)HPS_FLAG_STUCK_SET, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                list_misses(pending);
                break;
            }
            int here = lane;
            asm volatile("" : "+v"(here));             // this loop's lane arithmetic is not kept in registers from the start of the kernel
            const uint32_t v1 = pending ? ld_agent(sc + 2ull * set) : 0u;
            const bool busy = pending && (v1 & 1u);    // a writer holds the set: look again later
            shared_acquire();                          // the word is read before any key or row
            const int w = probe_wave<W, KPW, true>(K, key, set, pending && !busy, [] {}, lanes, here);
            const bool found = w >= 0;
            const uint64_t fmask = __ballot(found);
            if (here < 2) s_retry[wave][here] = 0u;
            if (found) {
                const int r = rank_in(fmask);
                s_src[wave][r] = (uint64_t)set * W + (uint32_t)w;
                s_dst[wave][r] = pos;
                s_set[wave][r] = set;
                s_v1[wave][r]  = v1;
                const uint32_t nf = (uint32_t)__popcll(fmask);
                if (kD && (nf & 1u) && r + 1 == (int)nf) {
                    s_src[wave][nf] = (uint64_t)set * W + (uint32_t)w;
                    s_dst[wave][nf] = pos;
                    s_set[wave][nf] = set;
                    s_v1[wave][nf]  = v1;
                }
            }
            wave_lds_fence();
            if (fmask)
                copy_rows_checked<(kD ? U : 8), kD>(g, V, out, &s_src[wave][0], &s_dst[wave][0], &s_set[wave][0],
                                                     &s_v1[wave][0], sc, (uint32_t)__popcll(fmask), &s_retry[wave][0], (uint32_t)here);
            wave_lds_fence();
            bool again = false;
            if (found) {
                const int r = rank_in(fmask);
                again = (s_retry[wave][r >> 5] >> (r & 31)) & 1u;
            }
            stamp(found && !again, w);
            list_misses(pending && !busy && !found);   // a clean miss is final
            pending = busy || again;
            wave_lds_fence();
            if (__ballot(pending)) __builtin_amdgcn_s_sleep(2);
        }
        wave_lds_fence();
        tell();
    }
}

// Query with in-tile deduplication (the paper deduplicates a batch before the lookup, Sec. 2.2;
// here each tile of WPB*64 positions does it in LDS).  An LDS hash table (2 slots per position,
// 64-bit compare-and-swap, linear probing) elects one representative position per distinct key of
// the tile.  Only representatives probe the cache and only their rows are read from memory; a
// row is then stored to the representative's position and to every duplicate position, which
// hang off the representative in an LDS linked list (atomic exchange on the list head).  Misses
// are reported per position as in query_kernel, and the helper wave does the same counter work.
template <int W, int U, int WPB>
__global__ void __launch_bounds__((WPB + 1) * kWave) query_dedup_kernel(const QueryArgs a) {
    constexpr int kTile = kWave * WPB;
    constexpr int kHash = 2 * kTile;
    static_assert((kHash & (kHash - 1)) == 0, "the LDS table is probed with a mask: its size must be a power of two");
    constexpr uint32_t kNil = 0xFFFFFFFFu;
    constexpr uint64_t kMissed = ~0ull;
    __shared__ unsigned long long h_key[kHash];
    __shared__ uint32_t h_own[kHash];
    __shared__ uint64_t r_slot[kTile];
    __shared__ uint32_t head[kTile];
    __shared__ uint32_t nxt[kTile];
    __shared__ uint64_t s_src[WPB][kWave];
    __shared__ uint32_t s_rep[WPB][kWave];
    __shared__ int64_t  s_mkey[WPB][kWave];
    __shared__ uint32_t s_mpos[WPB][kWave];
    __shared__ uint32_t s_wcnt[WPB];

    const int lane = lane_id();
    const int wave = (int)(threadIdx.x / kWave);
    const RowGeom g = a.g;
    const uint32_t rpi = (uint32_t)kWave >> g.lprShift;
    const uint32_t sub = (uint32_t)lane >> g.lprShift;
    const uint32_t cl  = (uint32_t)lane & (g.LPR - 1);

    for (uint32_t tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
        const uint32_t t  = tile / a.tiles_per_table;
        const uint32_t lt = tile - t * a.tiles_per_table;
        const uint32_t pos0 = t * a.B + lt * WPB * a.kpw;      // position of this tile's first key
        if (wave < WPB) {
            const Table   &tb   = a.tab[t];
            const uint32_t g_call = tb.T ? *tb.gdev + 1u : 0u;               // as in query_kernel
            const uint32_t tid  = (uint32_t)wave * a.kpw + (uint32_t)lane;   // index in the tile (idle lanes alias, unused)
            const uint32_t b    = lt * WPB * a.kpw + tid;
            const bool     inb  = lane < (int)a.kpw && b < a.B;
            const uint32_t pos  = pos0 + tid;
            const int64_t  key  = inb ? a.keys[pos] : kEmpty;
            const bool     live = inb && (!a.n_dev || b < *a.n_dev);
            const bool     want = live && !is_reserved(key);
            const uint64_t h    = mix64((uint64_t)key);
            const uint32_t hs   = (uint32_t)(h >> 32);
            const uint32_t set  = want ? (tb.smask ? (hs & tb.smask) : (hs % tb.S)) : 0u;

            for (uint32_t i = threadIdx.x; i < (uint32_t)kHash; i += kTile) h_key[i] = (unsigned long long)kEmpty;
            head[threadIdx.x] = kNil;
            __syncthreads();                                    // #1 table cleared

            bool is_rep = false;
            uint32_t my = 0;
            if (want) {
                uint32_t slot = (uint32_t)h & (kHash - 1);
                for (;;) {
                    const unsigned long long old =
                        atomicCAS(&h_key[slot], (unsigned long long)kEmpty, (unsigned long long)key);
                    if (old == (unsigned long long)kEmpty) { is_rep = true; h_own[slot] = tid; break; }
                    if (old == (unsigned long long)key) break;
                    slot = (slot + 1) & (kHash - 1);
                }
                my = slot;
            }
            __syncthreads();                                    // #2 representatives elected
            const uint32_t rep = is_rep ? tid : (want ? h_own[my] : tid);
            const int way = probe_wave<W, kWave>(tb.K, key, set, is_rep);
            if (is_rep) r_slot[tid] = way >= 0 ? (uint64_t)set * W + (uint32_t)way : kMissed;
            if (tb.T && is_rep && way >= 0) tb.T[(uint64_t)set * W + (uint32_t)way] = g_call;
            __syncthreads();                                    // #3 probe results visible
            const uint64_t res = want ? r_slot[rep] : kMissed;
            const bool hit = res != kMissed;

            const uint64_t missmask = __ballot(live && !hit);
            if (live && !hit) {
                const int r = rank_in(missmask);
                s_mpos[wave][r] = pos;
                s_mkey[wave][r] = key;
            }
            if (lane == 0) s_wcnt[wave] = (uint32_t)__popcll(missmask);

            if (hit && !is_rep) nxt[tid] = atomicExch(&head[rep], tid);     // join the representative's list
            const uint64_t repmask = __ballot(hit && is_rep);
            const uint32_t nh = (uint32_t)__popcll(repmask);
            if (hit && is_rep) {
                const int r = rank_in(repmask);
                s_src[wave][r] = res;
                s_rep[wave][r] = tid;
            }
            __syncthreads();                                    // #4 lists complete; helper starts

            const float *__restrict__ V = tb.V;
            for (uint32_t pass = 0; pass < g.passes; ++pass) {
                uint32_t chunk = cl + pass * g.LPR;
                chunk = chunk < g.C ? chunk : 0u;
                const uint32_t off = chunk * 4;
                for (uint32_t e0 = 0; e0 < nh; e0 += rpi * U) {
                    f32x4 buf[U];
                    uint32_t rp[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        uint32_t e = e0 + u * rpi + sub;
                        e = e < nh ? e : 0u;
                        rp[u] = s_rep[wave][e];
                        buf[u] = *reinterpret_cast<const f32x4 *>(V + s_src[wave][e] * g.d + off);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        __builtin_nontemporal_store(
                            buf[u], reinterpret_cast<f32x4 *>(a.out + (uint64_t)(pos0 + rp[u]) * g.d + off));
                        uint32_t p = head[rp[u]];
                        while (p != kNil) {                     // duplicate positions of this key
                            __builtin_nontemporal_store(
                                buf[u], reinterpret_cast<f32x4 *>(a.out + (uint64_t)(pos0 + p) * g.d + off));
                            p = nxt[p];
                        }
                    }
                }
            }
        } else {
            __syncthreads();
            __syncthreads();
            __syncthreads();
            __syncthreads();
            uint32_t total = 0;
#pragma unroll
            for (int w = 0; w < WPB; ++w) total += s_wcnt[w];
            uint64_t old = 0;
            if (lane == 0)
                old = __hip_atomic_fetch_add(a.slot, (1ull << 32) | (uint64_t)total, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
            old = (uint64_t)shfl64((int64_t)old, 0);
            uint32_t o = (uint32_t)old;
#pragma unroll
            for (int w = 0; w < WPB; ++w) {
                const uint32_t c = s_wcnt[w];
                for (uint32_t j = (uint32_t)lane; j < c; j += kWave) {
                    a.miss_idx[o + j]  = s_mpos[w][j];
                    a.miss_keys[o + j] = s_mkey[w][j];
                }
                o += c;
            }
            if ((uint32_t)(old >> 32) + 1u == a.n_tiles)
                finish_call(a.n_miss, a.slot, (uint32_t)lane < a.n_tables && a.tab[lane].T ? a.tab[lane].gdev : nullptr, (uint32_t)old + total, lane);
        }
        __syncthreads();                                        // #5 LDS is reused by the next tile
    }
}

// ------------------------------------------------------------------ insert / update

// What the writers need after their first loads; the rest they are given in registers, as query_kernel is.
struct WriteArgs {
    const float    *vals;
    float          *V;
    uint32_t       *T;
    uint32_t       *gdev;
    uint32_t       *flags;
    RowGeom         g;
};
typedef const __attribute__((address_space(4))) WriteArgs *WriteArgsIn;
constexpr uint32_t kWriteArgsAt = 56;          // behind 14 words
static_assert(alignof(WriteArgs) == 8, "kWriteArgsAt");
constexpr uint32_t kWriteGridX = 1u << 16;     // work-groups in a row of a writer's grid

// Replace (Alg. 3).  The first KPW lanes of a wave own one key each; all 64 lanes copy rows.  A
// pending lane takes its set's sequence word (the paper's slabset lock, Sec. 4.1) with one fetch-or
// of bit 0, which also reads the set's counter: it owns the set if the bit was clear.  The owners' sets
// are then searched with the wave-wide probe; new keys get their slot (key, counter, stamp) and row, and
// every owner lets go again: word + 2 if it changed the set, the old word if the key was already
// there.  Every lane also looks at its set without owning it: on the first attempt beside the fetch-or, before
// every further one in front of it, and a key that is found that way is done.
// No lane ever waits while the wave owns a set: each round every pending lane tries once, the owners'
// rows are copied by the whole wave, the sets are released, and the others try again.
// Bound by the chain of dependent round trips (key, word, set, rows, acknowledgement) in which a wave
// holds its sets; the owners' rows are therefore requested right behind their sets' keys, before it is known
// whether they are needed: 2^18 new rows of 512 bytes, inserted, updated and queried, 221 -> 208 us, 32,768 rows 18.5 ->
// 16.8 us per insert.  The first look keeps this from reading the rows of keys that are already there, in the round
// trip of the fetch-or: when it came in 2^18 such keys took 27.7 us, 47 without it (with the LRU policy 30 and 57), new
// ones 84-88 either way; now present ones take 19.7 (22.6), new ones 77 (90).  KPW = 16 or 8 (launch_write): four or eight times as many waves as keys / 64 share the row copies, and a
// wave's chain is two copy groups long, or one, instead of eight.
//
// Each policy has its own kernels, so that the victim counter's do not hold the LRU search's keys and stamps: in one kernel they took
// long rows from four waves per SIMD to three.  The LRU kernels of long rows keep four with kTight (up to 8 ways; it does not reach so far
// with more).  200,000 new rows of 1,280 / 2,048 bytes, 8 ways: counter 127 / 181 -> 117 / 174 us, LRU 125 / 163 -> 112 / 152.
// More than four waves fit short rows, but wait for each other's sets: 262,144 new keys over 2^11 sets of 8 ways 432 us with
// four, 505 with five; 64-way sets under LRU, where a search reads 768 bytes per key, 200,000 over 2^9 / 2^15 sets 3,750 / 150
// with three, 6,750 / 179 with four.
template <int W, int KPW, bool kLong, bool kLru>
__global__ void __attribute__((amdgpu_waves_per_eu(1, (W == 64 && kLru ? 3 : 4)))) __launch_bounds__(kBlock) insert_kernel(const u64x4 pointers, const u32x4 sizes, const uint64_t epochs, const WriteArgs) {
    constexpr bool kTight = kLong && kLru && W <= 8;
    __shared__ uint64_t s_dst[kWavesPerWg][kWave];
    __shared__ uint32_t s_srcrow[kWavesPerWg][kWave];
    __shared__ uint32_t s_first[kWavesPerWg * kWave];
    __shared__ int64_t  s_key[kWavesPerWg * KPW];
    __shared__ WriterGroup s_group;

    const int64_t *__restrict__ const keys = global_at<const int64_t>(pointers.x);
    const uint32_t *const n_dev = global_at<const uint32_t>(pointers.y);
    int64_t *const K = global_at<int64_t>(pointers.z);
    uint32_t *const sc = global_at<uint32_t>(pointers.w);
    const uint32_t S = sizes.y, smask = sizes.z;
    const int lane = lane_id();
    const int wave = wave_id();
    // One tile of KPW keys to a wave, no loop over tiles (see query_kernel).
    const uint32_t wg = blockIdx.y * kWriteGridX + blockIdx.x, first = (wg * kWavesPerWg + (uint32_t)wave) * KPW, i = first + lane;
    uint32_t n = sizes.x;
    if (n_dev) {
        const uint32_t nd = *n_dev;
        n = nd < n ? nd : n;
    }
    if ((uint64_t)wg * kWavesPerWg * KPW >= n) return;      // nothing for any wave of this work-group
    int64_t key = lane < KPW && i >= first && i < n ? keys[i] : kEmpty;
    WriteArgsIn in = (WriteArgsIn)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + kWriteArgsAt);
    asm volatile("" : "+s"(in));
    const float *const vals = in->vals;
    float *const V = in->V;
    const RowGeom g = {in->g.d, in->g.C, in->g.LPR, in->g.lprShift, in->g.passes, {in->g.c16.C, in->g.c16.packed}, {in->g.c8.C, in->g.c8.packed}};
    uint32_t *const pair = epoch_of(global_at<uint32_t>(epochs), wg);
    uint32_t *const T = in->T;
    const uint32_t g_now = kLru ? *in->gdev : 0u;           // Alg. 3 stamps with the current iteration count
    writer_enter(pair, &s_group);                           // its round trip runs beside that of the keys
    // Copies of a key among the first keys of the work-group: all of them write their number into the key's hash slot,
    // the one whose number stays carries the key, the others drop out (Alg. 3 ignores a key that is already there,
    // so only one copy can ever take effect).  A slot shared by different keys thins nothing.  Attempts on one set go one
    // after the other, 11 ns each, and with fewer keys per wave there are more of them: 16,384 keys with a key that
    // makes up a quarter of them 18.4 us with 16 keys per wave thinned wave by wave, 28.3 with 8, 12.1 this way; the barrier is
    // the one that writers have anyway.
    const uint32_t me = (uint32_t)(wave * KPW + lane);
    const uint32_t place = (uint32_t)(mix64((uint64_t)key) >> 8) % (uint32_t)(kWavesPerWg * kWave);
    if (!is_reserved(key)) {
        s_first[place] = me;
        s_key[me] = key;
    }
    __syncthreads();
    if (!is_reserved(key)) {
        const uint32_t o = s_first[place];
        if (o != me && s_key[o] == key) key = kEmpty;
    }
    bool told = wave != 0;                                  // only wave 0 has something to tell
    RowMover<(kLong ? 8 : 4), kLong> rows(g, vals, V, &s_srcrow[wave][0], &s_dst[wave][0]);

    bool pending = !is_reserved(key);
    const uint32_t set = pending ? set_of(key, S, smask) : 0u;

    // A search reads a set for every lane: the sets of those in m, for the others that of the first of them, which
    // costs no request.  (Lanes that are done reading their own sets once more, which others write to, took 262,144 new keys over
    // 2^14 sets from 130 to 148 us, over 2^16 from 88 to 97, and 70,000 under LRU of which a third are 64 keys from 38 to 58.)
    auto set_in = [&](bool in, uint64_t m) { return in ? set : (uint32_t)__builtin_amdgcn_readlane((int)set, __builtin_ctzll(m)); };
    uint32_t rounds = 0;
    while (const uint64_t pendmask = __ballot(pending)) {
        if (++rounds > kMaxRounds) {                             // a set never came free: skip these keys
            if (pending) __hip_atomic_fetch_or(in->flags, (uint32_t)HPS_FLAG_STUCK_SET, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
        // Look before owning: a key given many times (a miss list carries every occurrence) is found by
        // all but the first without taking the word, instead of each occurrence owning the set in turn.
        // On the first attempt the look travels beside the fetch-or, later in front of it.
        int seen = -1;
        int here = lane;
        if constexpr (kTight) asm volatile("" : "+v"(here));     // the searches' lane arithmetic is done again, not kept in registers
        if (rounds > 1) {
            seen = probe_wave<W, KPW, true>(K, key, set_in(pending, pendmask), pending, [] {}, KPW, here);
            if (pending && seen >= 0) {
                if (kLru) st_agent(T + (uint64_t)set * W + (uint32_t)seen, g_now);    // Alg. 3: refresh
                pending = false;
            }
        }
        // one 64-bit atomic on the set's {seq, ctr} word: takes the set and reads its counter
        uint64_t word = 1ull;
        if (pending)
            word = __hip_atomic_fetch_or(reinterpret_cast<uint64_t *>(seq_of(sc, set)), 1ull, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        if (rounds == 1) seen = probe_wave<W, KPW, true>(K, key, set_in(pending, pendmask), pending, [] {}, KPW, here);
        shared_acquire();                                        // the word is owned before the set is read
        writer_tell(&s_group, told);
        const uint32_t old = (uint32_t)word;
        const uint32_t c = (uint32_t)(word >> 32);
        bool own = pending && !(old & 1u);
        if (pending && seen >= 0) {
            if (kLru) st_agent(T + (uint64_t)set * W + (uint32_t)seen, g_now);
            if (own) st_agent(reinterpret_cast<uint64_t *>(seq_of(sc, set)), word);
            own = pending = false;
        }
        if (!__ballot(own)) {
            if (__ballot(pending)) __builtin_amdgcn_s_sleep(8);
            continue;
        }
        const uint64_t ownmask = __ballot(own);
        const int r = rank_in(ownmask);
        if (own) s_srcrow[wave][r] = i;
        wave_lds_fence();
        // the owners' rows are requested behind the sets' keys (LRU policy: and stamps) and travel while those are compared
        auto rows_too = [&] { rows.start((uint32_t)__popcll(ownmask)); };
        int victim = (int)(c & (W - 1));                         // victim counter
        int way;
        const uint32_t from = set_in(own, ownmask);
        if constexpr (kLru) way = probe_lru_wave<W, KPW, (kTight ? 1 : 4)>(K, T, key, from, own, g_now, victim, here, rows_too);
        else way = probe_wave<W, KPW, true>(K, key, from, own, rows_too, KPW, here);
        const bool fresh = own && way < 0;
        if (fresh) way = victim;
        if (kLru && own) st_agent(T + (uint64_t)set * W + (uint32_t)way, g_now);
        const uint64_t freshmask = __ballot(fresh);
        if (freshmask) {
            writer_entered(&s_group);
            if (fresh) st_agent(K + (uint64_t)set * W + (uint32_t)way, key);
            if (own) s_dst[wave][r] = fresh ? (uint64_t)set * W + (uint32_t)way : kSkipRow;
            wave_lds_fence();
            rows.finish(freshmask == ownmask);
        }
        wave_lds_fence();
        shared_release();                                        // rows and keys land before the words move on
        if (own) {
            // let go: a changed set gets seq + 2 and ctr + 1 in one store, an unchanged one its old word
            st_agent(reinterpret_cast<uint64_t *>(seq_of(sc, set)),
                     fresh ? (((uint64_t)(c + 1u) << 32) | (uint64_t)(old + 2u)) : word);
            pending = false;
        }
    }
    writer_leave(pair, &s_group, told);                              // (every hold that stored a key or a row ended with shared_release: they have landed)
}

// Update (Alg. 4) with one lock acquisition per run of lanes that share a set.  Key batches that
// come from a dump are in slot order: eight neighbouring keys belong to one set, and taking the
// set's word once per key would serialise them over eight rounds.  Here adjacent pending lanes
// with the same set form a group; the group's first lane reads the word and, if any lane of the
// group found its key, takes it once; all those lanes' rows are then written under that one hold.
// Two lanes of a group that found the same slot (a key given twice) are thinned to one per round.
// Lanes of different groups that meet on a set compete by compare-and-swap on its word; no lane
// waits while its wave owns a set.
// Bound by memory: 1 GiB of cached rows refreshed in dump order at 4.6 TB/s of rows read and written.  Four waves per
// SIMD (one GiB with its dump and query 438 us, 446 with the six that the registers would allow, on one device in turn;
// twice as many wave loads in flight: 2 us more there, 3 us more on 2^18 scattered rows).  Long rows of 16 and 32 ways need the limit from
// below too: with 129 registers 262,144 rows of 1,280 bytes, 32 ways, in a dump's order 145 us, 131 this way.
template <int W, int KPW, bool kLong>
__global__ void __attribute__((amdgpu_waves_per_eu(4, 4))) __launch_bounds__(kBlock) update_kernel(const u64x4 pointers, const u32x4 sizes, const uint64_t epochs, const WriteArgs) {
    __shared__ uint64_t s_dst[kWavesPerWg][kWave];
    __shared__ uint32_t s_srcrow[kWavesPerWg][kWave];
    __shared__ WriterGroup s_group;

    const int64_t *__restrict__ const keys = global_at<const int64_t>(pointers.x);
    const uint32_t *const n_dev = global_at<const uint32_t>(pointers.y);
    int64_t *const K = global_at<int64_t>(pointers.z);
    uint32_t *const sc = global_at<uint32_t>(pointers.w);
    const uint32_t S = sizes.y, smask = sizes.z;
    const int lane = lane_id();
    const int wave = wave_id();
    // One tile of KPW keys to a wave, no loop over tiles (see query_kernel).
    const uint32_t wg = blockIdx.y * kWriteGridX + blockIdx.x, first = (wg * kWavesPerWg + (uint32_t)wave) * KPW, i = first + lane;
    uint32_t n = sizes.x;
    if (n_dev) {
        const uint32_t nd = *n_dev;
        n = nd < n ? nd : n;
    }
    if ((uint64_t)wg * kWavesPerWg * KPW >= n) return;      // nothing for any wave of this work-group
    int64_t key = lane < KPW && i >= first && i < n ? keys[i] : kEmpty;
    WriteArgsIn in = (WriteArgsIn)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + kWriteArgsAt);
    asm volatile("" : "+s"(in));
    const float *const vals = in->vals;
    float *const V = in->V;
    const RowGeom g = {in->g.d, in->g.C, in->g.LPR, in->g.lprShift, in->g.passes, {in->g.c16.C, in->g.c16.packed}, {in->g.c8.C, in->g.c8.packed}};
    uint32_t *const pair = epoch_of(global_at<uint32_t>(epochs), wg);
    writer_enter(pair, &s_group);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);                      // (nobody waits in front of it for keys, with wave 0 also for its count)
    bool told = wave != 0;                                  // only wave 0 has something to tell

    bool pending = !is_reserved(key);
    const uint32_t set = pending ? set_of(key, S, smask) : 0u;

    uint32_t rounds = 0;
    while (const uint64_t pendmask = __ballot(pending)) {
        if (++rounds > kMaxRounds) {                             // a set never came free: skip these keys
            if (pending) __hip_atomic_fetch_or(in->flags, (uint32_t)HPS_FLAG_STUCK_SET, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
        // groups: maximal runs of adjacent pending lanes with equal set
        const uint32_t prev_set = (uint32_t)__shfl_up((int)set, 1, kWave);
        const int prev_pend = __shfl_up((int)pending, 1, kWave);
        const bool start = pending && (lane == 0 || !prev_pend || prev_set != set);
        const uint64_t startmask = __ballot(start);
        int here = lane;
        asm volatile("" : "+v"(here));                           // made here, not kept in registers beside the rows
        const uint64_t le_lane = ~0ull >> (63 - here);           // bits 0..lane
        const int leader = pending ? 63 - __builtin_clzll(startmask & le_lane) : lane;
        const uint64_t le_leader = leader == 63 ? ~0ull : ((2ull << leader) - 1);
        const uint64_t above = startmask & ~le_leader;
        const uint64_t lt_end = above ? ((1ull << __builtin_ctzll(above)) - 1) : ~0ull;
        const uint64_t gmask = pendmask & lt_end & ~(le_leader >> 1);    // lanes leader .. end-1 that are pending
        const bool is_leader = pending && lane == leader;

        uint32_t v = is_leader ? ld_agent(seq_of(sc, set)) : 0u;
        v = (uint32_t)__shfl((int)v, leader, kWave);
        const bool busy = pending && (v & 1u);
        shared_acquire();                                        // the word is read before the keys
        writer_tell(&s_group, told);
        // W lanes read a set's line, as in the other kernels; lanes without one to search read that of the first that has one, which
        // is read anyway.  With 64 keys to a wave each lane reads its own set instead where that is less work: in a dump's order, where
        // a run's lanes read the same line, and in wide sets when few lanes search, as behind a lost attempt.  (us, each lane its own / W lanes each /
        // this way.  Rows of 512 bytes, random order, 8 ways: 262,144 95 / 85 / 85, absent 15.5 / 9.5 / 9.5; 100,000 rows, 16 ways 88 / 75 / 72,
        // 64 ways 343 / 481 / 331, absent 37 / 21 / 22.  In a dump's order, 8 ways: 262,144 51.6 / 50.0 / 49.1; 100,000, 16 ways 29.0 / 29.1 / 27.1, 64 ways
        // 39 / 62 / 39.  Both searches in the kernels of long rows and 8 ways cost 0.3-1 us in every order: 65,536 of 1,280 bytes in a dump's
        // 34.7 / 34.9 / 35.1, random 53.6 / 53.5 / 54.4; fewer than four ways gain nothing.  With 16 keys to a wave W lanes each throughout.)
        const bool search = pending && !busy;
        const uint64_t searchmask = __ballot(search);
        constexpr bool kBoth = KPW == kWave && W >= (kLong ? 16 : 4);
        constexpr int kFew = W == 64 ? 32 : W >= 16 ? 8 : 0;
        int way = -1;
        if (kBoth && (2 * __popcll(startmask) <= __popcll(pendmask) || __popcll(searchmask) <= kFew)) {
            if (search) {
                constexpr int F = W > 32 ? 32 : W;               // keys in flight together
#pragma unroll 1
                for (int w0 = 0; w0 < W; w0 += F) {
                    int64_t sk[F];
#pragma unroll
                    for (int w = 0; w < F; ++w) sk[w] = ld_agent(K + (uint64_t)set * W + w0 + w);
#pragma unroll
                    for (int w = 0; w < F; ++w)
                        if (sk[w] == key) way = w0 + w;
                }
            }
        } else if (searchmask) {
            const uint32_t some = (uint32_t)__builtin_amdgcn_readlane((int)set, __builtin_ctzll(searchmask));
            way = probe_wave<W, KPW, true>(K, key, search ? set : some, search);
        }
        if (search && way < 0) pending = false;                  // not cached: ignored
        bool winner = search && way >= 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {                            // one lane per slot and round
            const uint64_t m = __ballot(winner && way == w) & gmask;
            if (winner && way == w && lane != __builtin_ctzll(m)) winner = false;
        }
        const bool group_needs = (__ballot(winner) & gmask) != 0;
        bool won = false;
        if (is_leader && !busy && group_needs) {
            uint32_t expect = v;
            won = __hip_atomic_compare_exchange_strong(seq_of(sc, set), &expect, v + 1u, __ATOMIC_RELAXED,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const bool gwon = __shfl((int)won, leader, kWave) != 0;
        const bool act = winner && gwon;
        const uint64_t actmask = __ballot(act);
        if (actmask) {
            shared_acquire();
            writer_entered(&s_group);
            if (act) {
                const int r = rank_in(actmask);
                uint32_t at = first;
                asm volatile("" : "+s"(at));                     // i, made again for the same reason
                s_dst[wave][r] = (uint64_t)set * W + (uint32_t)way;
                s_srcrow[wave][r] = at + (uint32_t)lane;
            }
            wave_lds_fence();
            copy_rows_shared<(kLong ? 8 : 4), kLong>(g, vals, V, &s_srcrow[wave][0], &s_dst[wave][0], (uint32_t)__popcll(actmask));
            wave_lds_fence();
            shared_release();                                    // rows land before the word moves on
            if (won) st_agent(seq_of(sc, set), v + 2u);
            if (act) pending = false;
        }
    }
    writer_leave(pair, &s_group, told);
}

// ------------------------------------------------------------------ small kernels

__global__ void set_u32_kernel(uint32_t *p, uint32_t v) { *p = v; }

__global__ void fill_keys_kernel(int64_t *K, uint64_t n, int64_t v) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        K[i] = v;
}

// Export / import of the victim counters: ctr[s] <-> the upper half of the set's {seq, ctr} word.
// An import leaves every sequence word at zero (no writer, nothing in flight).
__global__ void counters_out_kernel(const uint32_t *sc, uint64_t S, uint32_t *ctr) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < S;
         i += (uint64_t)gridDim.x * blockDim.x)
        ctr[i] = sc[2 * i + 1];
}
// (an import replaces the state: no writer holds a set of it, and none has counted itself in)
__global__ void counters_in_kernel(uint32_t *sc, uint64_t S, const uint32_t *ctr, uint32_t *epoch) {
    if (blockIdx.x == 0 && threadIdx.x < 2 * kEpochs) epoch[threadIdx.x / 2 * kEpochStride + threadIdx.x % 2] = 0u;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < S;
         i += (uint64_t)gridDim.x * blockDim.x) {
        sc[2 * i] = 0u;
        sc[2 * i + 1] = ctr[i];
    }
}

// hps_cache_debug_set_seq.  A writer that holds a set (odd word) has counted itself in and not yet out; writers that
// are at work count on the same pair.
__global__ void set_seq_kernel(uint32_t *seq, uint32_t value, uint32_t *epoch) {
    const uint32_t old = __hip_atomic_exchange(seq, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((old ^ value) & 1u) __hip_atomic_fetch_add(epoch + (value & 1u ? 0 : 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Dump (Sec. 4.2): compact the non-empty keys of a slot range.  A work-group takes a tile of
// 256*KPT consecutive slots, keeps KPT keys per lane in registers, and needs one counter atomic
// per tile (same counter-word scheme as query).  The output keeps slot order inside a tile, so the
// keys of one set stay next to each other: an Update over the dumped keys then takes each set once
// for all its keys (update_kernel groups such runs) and writes the rows of a set, which are
// contiguous in memory, together.
template <int KPT>
__global__ void __launch_bounds__(kBlock) dump_kernel(const int64_t *__restrict__ K, uint64_t first,
                                                      uint64_t n_slots, int64_t *keys_out,
                                                      uint32_t *n_out, uint64_t *slot,
                                                      uint32_t n_tiles) {
    constexpr uint32_t kTileSlots = kBlock * KPT;
    constexpr int kCnt = KPT * kWavesPerWg;                // one count per (j, wave)
    static_assert(kCnt <= kBlock, "the count scan gives every count its own thread");
    __shared__ uint32_t s_cnt[kCnt];                       // [j][wave] counts, then exclusive prefixes
    __shared__ uint32_t s_wtot[kWavesPerWg];
    __shared__ uint32_t s_base;
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x / kWave);
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        int64_t key[KPT];
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const uint32_t q = (uint32_t)j * kBlock + threadIdx.x;
            const uint64_t i = (uint64_t)tile * kTileSlots + q;
            key[j] = i < n_slots ? __builtin_nontemporal_load(K + first + i) : kEmpty;     // read once
        }
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const uint64_t m = __ballot(key[j] != kEmpty);
            if (lane == 0) s_cnt[j * kWavesPerWg + wave] = (uint32_t)__popcll(m);
        }
        __syncthreads();
        // exclusive scan of the kCnt counts over the work-group: inside each wave, then across waves
        const uint32_t c = threadIdx.x < (uint32_t)kCnt ? s_cnt[threadIdx.x] : 0u;
        uint32_t incl = c;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t up = (uint32_t)__shfl_up((int)incl, o, kWave);
            if (lane >= o) incl += up;
        }
        if (lane == kWave - 1) s_wtot[wave] = incl;
        __syncthreads();
        uint32_t woff = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kWavesPerWg; ++w) {
            const uint32_t t = s_wtot[w];
            if (w < wave) woff += t;
            total += t;
        }
        if (threadIdx.x < (uint32_t)kCnt) s_cnt[threadIdx.x] = woff + incl - c;
        if (threadIdx.x == 0) {
            const uint64_t old = __hip_atomic_fetch_add(slot, (1ull << 32) | (uint64_t)total,
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_base = (uint32_t)old;
            if ((uint32_t)(old >> 32) + 1u == n_tiles) {
                *n_out = (uint32_t)old + total;
                __hip_atomic_store(slot, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        const uint32_t base = s_base;
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const uint64_t m = __ballot(key[j] != kEmpty);
            if (key[j] != kEmpty)
                __builtin_nontemporal_store(key[j], keys_out + base + s_cnt[j * kWavesPerWg + wave] + (uint32_t)rank_in(m));
        }
        __syncthreads();
    }
}

// Lower-tier stand-in.  A wave makes up to 32 rows at a time (rows of 16 bytes: 64), LPR lanes to a row, four consecutive
// elements per lane and pass: the inner mix, which depends on the element and not on the key, is made
// once per lane and pass instead of once per element.  Bound by the 64-bit products of the mixes (four
// per element before, two now) and by the rows written: 31.7 -> 20.7 us for the 90,000 missing rows of a
// 425,984-key batch, written twice.  Few rows are spread over all waves (7,400 rows in 32s: 6.5 us, spread 4.1 us).
// kPast: rows that go to both places.  The compact copy is what the caller reads next (an insert of the missing rows), the other
// goes past the caches (streaming step of 425,984 keys 108.6 -> 106.0 us).
constexpr uint32_t kBackingRows  = 32;
constexpr uint32_t kBackingWaves = 8192;         // as many as 256 CUs hold
template <bool kPast>
__global__ void __launch_bounds__(kBlock) backing_kernel(const int64_t *__restrict__ keys, uint32_t n,
                                                         const uint32_t *__restrict__ n_dev, uint32_t version, const RowGeom g,
                                                         float *rows, const uint32_t *__restrict__ scatter_idx,
                                                         float *scatter_out) {
    if (n_dev) {
        const uint32_t nd = *n_dev;
        n = nd < n ? nd : n;
    }
    const uint32_t lane = (uint32_t)lane_id();
    const uint32_t sub = lane >> g.lprShift;                 // which row of a wave store this lane serves
    const uint32_t rpi = (uint32_t)kWave >> g.lprShift;
    uint32_t per = n / kBackingWaves + 1u;
    per = per < rpi ? rpi : per < kBackingRows ? per : kBackingRows;
    // a wave takes one pass of a tile at a time: few long rows are shared by many waves (100 rows of 16 KiB 9.4 -> 5.5 us)
    const uint64_t units = ((uint64_t)n + per - 1) / per * g.passes, step = (uint64_t)gridDim.x * kWavesPerWg;
    for (uint64_t u = (uint64_t)blockIdx.x * kWavesPerWg + wave_id(); u < units; u += step) {
        const uint64_t i0 = u / g.passes * per;
        const uint32_t cnt = n - i0 < per ? (uint32_t)(n - i0) : per;
        const int64_t key = lane < cnt ? keys[i0 + lane] : 0;
        const uint32_t to = scatter_idx && lane < cnt ? scatter_idx[i0 + lane] : 0u;
        const uint32_t c = (lane & (g.LPR - 1u)) + (uint32_t)(u % g.passes) * g.LPR;   // all lanes stay: each holds a key that others ask it for
        uint64_t inner[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            inner[e] = mix64((((uint64_t)version << 32) | (c * 4u + (uint32_t)e)) + 0x9E3779B97F4A7C15ull);
        for (uint32_t r0 = 0; r0 < cnt; r0 += rpi) {
            const uint32_t r = r0 + sub;
            const uint64_t k = (uint64_t)shfl64(key, (int)r);            // r < 64; lanes past cnt store nothing
            const uint32_t w = (uint32_t)__shfl((int)to, (int)r, kWave);
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t z = mix64(k ^ inner[e]);
                x[e] = (float)((int32_t)(z >> 40) - (1 << 23)) * 0x1.0p-23f;   // exact: 24-bit integer * 2^-23
            }
            if (r < cnt && c < g.C) {
                const f32x4 v4 = {x[0], x[1], x[2], x[3]};
                if (rows) *reinterpret_cast<f32x4 *>(rows + (i0 + r) * g.d + c * 4) = v4;
                f32x4 *const to_out = reinterpret_cast<f32x4 *>(scatter_out + (uint64_t)w * g.d + c * 4);
                if (kPast) __builtin_nontemporal_store(v4, to_out);
                else if (scatter_idx) *to_out = v4;
            }
        }
    }
}

// out[i] = rows[inverse[i]] (hps_expand_rows): a wave takes kpw neighbouring positions and moves their
// rows as the query does, all of them in flight before its first store.  Bound by memory: 106,496 positions over 47,000
// rows of 512 bytes (79 MB) 17.6 us with four rows per group of lanes and step, 16.9 with the query's copy, 16.0 without its conditions.
template <int U, int WPB, int kD>
__global__ void __launch_bounds__(WPB * kWave) expand_rows_kernel(const float *__restrict__ rows, const uint32_t *__restrict__ inverse,
                                                                  uint32_t n, uint32_t kpw, const RowGeom g, float *__restrict__ out) {
    __shared__ uint32_t s_src[WPB][kWave];
    __shared__ uint32_t s_dst[WPB][kWave];
    const uint32_t lane = (uint32_t)lane_id();
    const int wave = wave_id();
    const uint64_t pos0 = ((uint64_t)blockIdx.x * WPB + wave) * kpw;
    if (pos0 >= n) return;
    const uint32_t cnt = n - pos0 < kpw ? (uint32_t)(n - pos0) : kpw;
    if (lane < cnt + (kD ? cnt & 1u : 0u)) {                 // a copy of the last entry behind an odd number of them (less than 64)
        const uint32_t p = (uint32_t)pos0 + (lane < cnt ? lane : cnt - 1u);
        s_src[wave][lane] = inverse[p];
        s_dst[wave][lane] = p;
    }
    wave_lds_fence();
    copy_rows<U, kD>(g, rows, out, &s_src[wave][0], &s_dst[wave][0], cnt, [] {});
}

// ------------------------------------------------------------------ measurement kernels (hps_membench.h)

// The row movement of query_kernel's plain variant alone: same tile shape, same copy loop, but the
// source slot of every position is given, so nothing is hashed, probed or compacted.
template <int U, int WPB, int kD>
__global__ void __launch_bounds__(WPB * kWave) membench_gather_kernel(const float *__restrict__ rows,
                                                                      const uint32_t *__restrict__ slot_of, uint32_t n,
                                                                      uint32_t kpw, const RowGeom g, float *__restrict__ out) {
    __shared__ uint32_t s_src[WPB][kWave];
    __shared__ uint32_t s_dst[WPB][kWave];
    const int lane = lane_id();
    const int wave = (int)(threadIdx.x / kWave);
    const uint32_t pos = (blockIdx.x * WPB + wave) * kpw + lane;
    const bool inb = lane < (int)kpw && pos < n;
    const uint32_t sl = inb ? slot_of[pos] : 0xFFFFFFFFu;
    const bool hit = sl != 0xFFFFFFFFu;
    const uint64_t hitmask = __ballot(hit);
    const uint32_t nh = (uint32_t)__popcll(hitmask);
    if (hit) {
        const int r = rank_in(hitmask);
        s_src[wave][r] = sl;
        s_dst[wave][r] = pos;
        if (kD && (nh & 1u) && r + 1 == (int)nh) {          // (an odd number is less than 64)
            s_src[wave][nh] = sl;
            s_dst[wave][nh] = pos;
        }
    }
    wave_lds_fence();
    if (nh) copy_rows<U, kD>(g, rows, out, &s_src[wave][0], &s_dst[wave][0], nh, [] {});
}

// Half of that row movement: kReads = true issues the group's row loads and stores nothing (the
// loaded words are folded into one value that is stored only if it equals a constant the data never
// produces, so the loads stay); kReads = false stores a register pattern to the same destination
// rows and loads nothing.  Work distribution, group size and access width are copy_rows'.
template <int U, int WPB, bool kReads>
__global__ void __launch_bounds__(WPB * kWave) membench_half_kernel(const float *__restrict__ rows,
                                                                    const uint32_t *__restrict__ slot_of, uint32_t n,
                                                                    uint32_t kpw, float *__restrict__ out) {
    __shared__ uint32_t s_src[WPB][kWave];
    __shared__ uint32_t s_dst[WPB][kWave];
    const uint32_t lane = (uint32_t)lane_id();
    const int wave = (int)(threadIdx.x / kWave);
    const uint32_t pos = (blockIdx.x * WPB + wave) * kpw + lane;
    const bool inb = lane < kpw && pos < n;
    const uint32_t sl = inb ? slot_of[pos] : 0xFFFFFFFFu;
    const bool hit = sl != 0xFFFFFFFFu;
    const uint64_t hitmask = __ballot(hit);
    const uint32_t cnt = (uint32_t)__popcll(hitmask);
    if (hit) {
        const int r = rank_in(hitmask);
        s_src[wave][r] = sl;
        s_dst[wave][r] = pos;
    }
    wave_lds_fence();
    const uint32_t sub = lane >> 5, off = (lane & 31u) * 4u;            // 512-byte rows: 32 lanes per row, 2 rows per wave load
    for (uint32_t e0 = 0; e0 < cnt; e0 += 2 * U) {
        f32x4 buf[U];
        uint32_t ent[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t e = e0 + 2 * u + sub;
            ent[u] = e < cnt ? e : 0xFFFFFFFFu;
            if (kReads) buf[u] = *reinterpret_cast<const f32x4 *>(rows + (uint64_t)s_src[wave][e < cnt ? e : 0u] * 128 + off);
            else        buf[u] = f32x4{(float)lane, (float)u, (float)e, 1.0f};
        }
        if (kReads) {
            __builtin_amdgcn_s_waitcnt(0x0F70);
            f32x4 acc = buf[0];
#pragma unroll
            for (int u = 1; u < U; ++u) acc += buf[u];
            if (acc.x == 1.2345678e-30f && acc.y == acc.x) out[0] = acc.z;     // never true for the backing rows
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (ent[u] != 0xFFFFFFFFu)
                    __builtin_nontemporal_store(buf[u], reinterpret_cast<f32x4 *>(out + (uint64_t)s_dst[wave][ent[u]] * 128 + off));
        }
    }
}

template <int U, bool kNT>
__global__ void __launch_bounds__(kBlock) membench_copy_kernel(const f32x4 *__restrict__ src, f32x4 *__restrict__ dst, uint64_t n16) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    for (; i + (U - 1) * stride < n16; i += U * stride) {
        f32x4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = kNT ? __builtin_nontemporal_load(src + i + u * stride) : src[i + u * stride];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kNT) __builtin_nontemporal_store(x[u], dst + i + u * stride);
            else dst[i + u * stride] = x[u];
        }
    }
    for (; i < n16; i += stride) dst[i] = src[i];
}

// ------------------------------------------------------------------ host side

RowGeom make_geom(uint32_t d) {
    RowGeom g;
    g.d = d;
    g.C = d / 4;
    uint32_t lpr = 1, sh = 0;
    while (lpr < g.C && lpr < (uint32_t)kWave) { lpr <<= 1; ++sh; }
    g.LPR = lpr;
    g.lprShift = sh;
    g.passes = (g.C + lpr - 1) / lpr;
    auto step = [](uint32_t C) {               // lane * (inv * C - 2^16) < 2^16 for lane, C <= 64: the quotient is exact
        const uint32_t inv = C > (uint32_t)kWave ? 0u : (65536u + C - 1) / C;
        return ChunkStep{C, inv | ((uint32_t)kWave / C) << 17 | ((uint32_t)kWave % C) << 24};
    };
    g.c16 = step(g.C);
    g.c8 = step(d / 2);
    return g;
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

}  // namespace

struct hps_cache {
    uint64_t magic;
    int      device;
    uint64_t S;
    uint32_t W, d;
    int64_t  *K;
    float    *V;
    uint32_t *sc;                         // [S][2]: {sequence word, victim counter}
    uint64_t *ring;                       // 2 * kRing counter words, all zero between calls
    std::mutex word_mu;
    std::unordered_map<void *, uint32_t> word_of_stream;
    uint32_t word_half;                   // which half of `ring` is being handed out
    std::atomic<int> concurrent_writers;
    std::atomic<int> query_dedup;
    int      policy;                      // HPS_POLICY_*
    uint32_t *T;                          // access stamps (LRU policy), else nullptr
    uint32_t *epoch;                      // kEpochs {started, finished} pairs of writer work-groups
    uint32_t *flags;                      // device words: [0] HPS_FLAG_* bits, [1] g, the global iteration
                                          // count of Alg. 2 (one step per query call, LRU policy)
    int      n_cus;                       // compute units of the device
};

namespace {

hps_status_t check_handle(const hps_cache *c) {
    if (!c || c->magic != kMagic) return fail(HPS_ERR_INVALID_ARG, "invalid cache handle");
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != c->device)
        return fail(HPS_ERR_INVALID_ARG, "cache was created on device " + std::to_string(c->device) +
                                             " but device " + std::to_string(dev) + " is current");
    return HPS_OK;
}

Table table_of(const hps_cache *c) {
    Table t;
    t.K = c->K;
    t.V = c->V;
    t.sc = c->sc;
    t.S = (uint32_t)c->S;
    t.smask = (c->S & (c->S - 1)) == 0 ? (uint32_t)(c->S - 1) : 0u;
    if (c->S == 1) t.smask = 0;           // S = 1: "h % 1" = 0 (a zero mask means "use modulo")
    t.T = c->T;
    t.gdev = c->flags + 1;
    t.flags = c->flags;
    t.epoch = c->epoch;
    return t;
}

// Counter word of query/dump calls on `stream`.  Calls on one stream run one after the other and
// each leaves its word at zero, so they can share one; calls on different streams may overlap and
// get different words.  The pool is two halves of kRing words: streams are given words of the
// current half in order of first sight; when a half is used up (kRing different stream handles,
// e.g. a caller that keeps creating streams) the table is forgotten and the other half is
// handed out, so a kernel still running with a word of the old half is never disturbed.
// A kernel captured into a graph keeps the word of the stream it was captured on.
uint64_t *counter_word(hps_cache *c, void *stream) {
    std::lock_guard<std::mutex> lk(c->word_mu);
    auto it = c->word_of_stream.find(stream);
    if (it == c->word_of_stream.end()) {
        if (c->word_of_stream.size() >= kRing) {
            c->word_of_stream.clear();
            c->word_half ^= 1u;
        }
        it = c->word_of_stream.emplace(stream, c->word_half * kRing + (uint32_t)c->word_of_stream.size()).first;
    }
    return c->ring + it->second;
}

// Launch shape of the query kernel: wpb worker waves per work-group, kpw keys per worker wave, row
// copy in groups of u wave loads.  All figures are us per launch on 256 CUs (checked / plain where both are given).
//
// Keys per wave: 16 KiB of rows (64 rows of up to 256 bytes) while the batch fits the CUs that way, else up to 32 KiB, which is the
// longest group.  Fewer and larger waves than would fill the chip: every tile adds to one counter word, ~11 ns each
// one after the other (26,624 keys of 512 bytes 15 / 32 keys to a wave 8.4 / 7.5, of 256 bytes 15 / 64 8.1 / 6.9; 106,496 keys 60 / 64
// 16.1 / 15.6).  Small batches are bound by the chain of round trips of a wave, to which its own rows add, and go down to 8 keys (16 from 4,096 keys on), for about
// 100 tiles (4,907 keys plain 12 / 16 keys to a wave, of 512 bytes 4.8 / 4.6, of 128 bytes 4.6 / 4.4).
// Beyond one round of tiles over the CUs the waves are trimmed such that the last round is full (106,496 keys of 1 KiB 64 / 32 to a wave 34.8 / 30);
// with several tables the keys per wave go up as long as the tables' last, partly empty tiles would start another round (26 x 1,024 keys checked
// 16.1 -> 11.2), and where they would with full waves too, the waves are trimmed for one round more (26 x 4,096 plain 18.5 -> 15.5, 7 x 16,384 18.5 -> 15.6; rows of more than 256 bytes: of shorter ones a CU holds several work-groups).
//
// Workers.  4 while that makes few tiles, 5 up to three quarters of the CUs, then 7 (5 / 7 / 8, 26,624 keys of 512 bytes 7.5 / 7.8 / 7.9;
// 7 / 8, 106,496 keys 15.6 / 15.8, 425,984 keys 58.2 / 60.2, 106,496 of 1 KiB 29.9 / 30.7).  From 2^19 rows of up to 256 bytes on 11, one work-group per CU
// (7 / 11, checked: 851,968 rows of 256 bytes 72 / 67.5, of 128 bytes 44.5 / 43.1, of 64 bytes 32.8 / 32.2; at 425,984 rows of 128 bytes 23.3 / 23.5), plain of up to 32
// bytes 15 (11 / 15, 3,407,872 of 16 bytes 74.6 / 68.0); sets of more than 16 ways not, whose keys spill there.  Plain, short rows from where tiles of 7 x 64 keys
// are more than the CUs: of up to 128 bytes 15 or 11, whichever takes fewer rounds, with 64 keys to a wave, since two or three work-groups fit a CU (7 trimmed / this way, 118,205 keys
// of 128 bytes 11.3 / 8.3, 261,863 15.4 / 12.2, 475,504 22.5 / 19.1; of 64 bytes 389,757 18.7 / 13.6; 2 tables x 59,029 11.2 / 8.4), of up to 256 bytes 11 for one round (118,205 keys
// 12.0 / 10.1).  Over several rounds their waves are trimmed as well, to 48 keys at least (64 / trimmed, rows of 128 bytes that come from 2 GiB of memory: 286,000 keys 17.2 / 16.3, 364,000 21.5 / 19.3, 425,984 22.8 / 21.7,
// from the caches 370,000 20.2 / 20.0).  A length on the device, rows of 512 bytes plain: 8 where that is one round and 7 are two (59,000 of 118,587 keys 12.4 / 9.6).
//
// Sets of 32 and 64 ways: a wave reads them for 16 or 8 lanes at a time, a wave load for two keys or one, so its keys are whole 16s or 8s while the batch fits the CUs, of 64 ways
// 24 at most, and half the CUs get a tile (20,214 keys of 128 bytes plain, 32 ways 49 / 32 keys to a wave 7.3 / 6.4, 64 ways 49 / 24 9.6 / 7.5; 8,192 of 512 bytes, 32 ways 20 / 16 6.0 / 5.6).  Not more than 16 KiB of rows
// for it (6 tables x 4,481 keys of 400 bytes, 32 ways 48 / 32 11.3 / 9.8), and rows of more than 1 KiB as in other sets (16,282 keys of 2 KiB, 64 ways 16 / 10 15.5 / 13.2).
//
// Group size: a wave's whole share of rows in one group (a second group waits, with its own loads, for the
// first group's stores), and not much more: the registers of a larger group are waves that the CU cannot
// hold, and its code, all of it executed, lines that a short launch has to fetch (13,312 keys of 512 bytes in groups of 16 / 32
// 6.35 / 6.30, 5,000 keys in groups of 8 / 16 6.1 / 6.2; 425,984 keys in groups of 32 / 16 58 / 70).  11 workers with rows of 128 bytes: 16 / 8 43.1 / 44.2.
//
// A length on the device: `deal` neighbouring keys go to a wave at a time, sixteen (a line of the batch; 50,000 of 106,496 keys in fours / sixteens 16.2 / 12.3,
// 47,000 9.3 / 8.9) or as many as have 16 KiB of rows, since sixteen more or less are what one wave has more than another (sixteens / this way,
// 33,000 of 41,033 keys of 4 KiB 38.1 / 33.1, of 2 KiB 21.2 / 19.3) or all that a wave has (820 of 4 KiB 12.7 / 6.0).  Of rows of 2 KiB and more a deal has 8 KiB: a wave with two of
// 16 KiB beside one with three waits for it (16 / 8 KiB, 22,937 of 32,768 keys of 2 KiB 18.7 / 16.4, 11,468 of 16,384 of 4 KiB 18.4 / 16.2; a fifth of them 8.0 / 8.8).  A wave's keys are whole deals, so that they
// stay one group of rows (19,000 of 24,137 keys of 768 bytes plain, 21 keys to a wave 9.2, 16 7.6).  Over several rounds sixteens are the faster ones
// again (24,000 of 118,587 keys of 1,280 bytes plain in eights / sixteens 12.6 / 9.8).
struct QueryShape { uint32_t kpw; int u, wpb; uint32_t deal; };
uint32_t deal_of(uint32_t d) {
    uint32_t k = 16;
    while (k > 1 && (uint64_t)k * d * 4 > (d < 512 || k == 2 ? 16384 : 8192)) k >>= 1;
    return k;
}

// Most rows of d words that a wave moves with copy_rows, which counts their 16-byte chunks in 32 bits (fewer than 64
// only for rows of 512 MiB and more).
uint64_t most_rows(uint32_t d) { return (1ull << 31) / (d / 4); }

QueryShape query_shape(uint32_t n_tables, uint64_t batch, uint32_t d, uint64_t cus, bool coherent, bool dedup, uint32_t ways = 8, bool n_dev = false) {
    const uint64_t n = n_tables * batch, row = (uint64_t)d * 4;
    // a tile holds keys of one table: with several tables their last tiles are not full
    auto tiles_of = [&](uint64_t keys) { return n_tables * ((batch + keys - 1) / keys); };
    auto rounds_of = [&](uint64_t workers) { return (tiles_of(workers * kWave) + cus - 1) / cus; };     // with 64 keys to a wave
    auto rows_of = [&](uint64_t bytes) {                       // rows of a wave
        const uint64_t k = bytes / row;
        return k < kMinKeysPerWave ? (uint64_t)kMinKeysPerWave : k < (uint64_t)kWave ? k : (uint64_t)kWave;
    };
    uint64_t deal = !n_dev || dedup ? 1 : deal_of(d);
    auto whole = [&](uint64_t k) { return (k + deal - 1) / deal * deal; };
    const uint64_t block = ways > 16 && !dedup && d <= 256 ? 512 / ways : 1;       // lanes that the probe searches or leaves out together
    uint64_t some = rows_of(16384);
    if (block == 8 && some > 24) some = 24;
    const uint64_t most = dedup || n_dev ? (uint64_t)kWave : rows_of(32768);
    QueryShape q{(uint32_t)most, 0, 0, 0};
    const bool small = !dedup && d <= 64, many = small && ways <= 16 && n >= (n_dev ? 1u << 18 : 1u << 19);
    const bool between = small && !many && !coherent && rounds_of(7) > 1 && (ways > 16 ? ways == 32 && rounds_of(7) == 2 : d <= 32 || rounds_of(11) == 1);
    if (dedup) q.wpb = n < (1u << 14) ? 4 : 8;
    else if (many) q.wpb = d <= 8 && !coherent ? 15 : 11;
    else if (between) q.wpb = ways > 16 ? 7 : d <= 32 && rounds_of(15) < rounds_of(11) ? 15 : 11;
    else if (n_dev && !coherent && d == 128 && rounds_of(7) == 2 && rounds_of(8) == 1) q.wpb = 8;
    else q.wpb = n <= 2 * some * cus ? 4 : 4 * n <= 15 * some * cus ? 5 : 7;      // up to cus / 2 and 3 / 4 cus tiles of that many keys per wave
    const uint64_t full = (uint64_t)q.wpb * most * cus;        // keys per round
    uint64_t rounds = n ? (n + full - 1) / full : 1;
    if (!dedup && d > 64 && q.wpb == 7 && rounds < 8 && tiles_of(7 * most) > rounds * cus) ++rounds;
    if (rounds <= 8 && (!between || (rounds > 1 && ways <= 16))) {
        uint64_t k = (n + q.wpb * cus * rounds - 1) / (q.wpb * cus * rounds);
        if (between && k < 48) k = 48;
        if (coherent) k += k / 15;                             // (a few CUs without a tile are less than the tiles more; 425,984 keys plain 60 / 64 56.1 / 57.4)
        if (rounds == 1) {
            uint64_t least = dedup ? kMinKeysPerWave : ((block > 1 ? 4 : 5) * n + 2 * q.wpb * cus - 1) / (2 * q.wpb * cus);      // 1 / 2 or 2 / 5 cus tiles
            if (n >= 4096 && (dedup || least < 16)) least = 16;
            if (least > some) least = some < 16 ? some : some - some % deal;
            if (least < kMinKeysPerWave) least = kMinKeysPerWave;
            if (least > block) {
                least = (least + block / 2) / block * block;
                if (least > some && some >= block) least = some - some % block;
            }
            if (k < least) k = least;
            if (block == 8) k = (k + 7) / 8 * 8;
            if (row > 512 && k > least) {
                if (deal > 8 && whole(k) * row > 32768) deal = 8;
                k = whole(k);
            }
        } else if (deal > 1) deal = 16;
        while (n_tables > 1 && k < (q.wpb < 7 ? some : most) && tiles_of(q.wpb * k) > rounds * cus) ++k;
        if (k < most) q.kpw = (uint32_t)k;
    }
    if (!dedup && q.kpw > most_rows(d)) q.kpw = (uint32_t)most_rows(d);
    if (deal > 1 && (q.kpw >= 16 || q.kpw % deal == 0)) q.deal = (uint32_t)deal;
    const uint64_t bytes = (q.deal ? whole(q.kpw) : q.kpw) * row;      // a wave's rows
    if (d == 128 && q.wpb == 4 && q.kpw <= 8) q.u = 4;
    else if (q.wpb == 11) q.u = d <= (between ? 32u : 16u) ? 8 : 16;
    else if (q.wpb == 8 && !dedup) q.u = 32;
    else q.u = bytes <= 8192 && (d != 128 || q.wpb == 4) ? 8 : bytes <= 16384 ? 16 : 32;
    return q;
}

template <int W, int U, int WPB, bool kCoherent, int kD>
void launch_query_kernel(const QueryArgs &a, bool full, hipStream_t st) {
    const dim3 grid(a.n_tiles < kGridX ? a.n_tiles : kGridX, (a.n_tiles + kGridX - 1) / kGridX), block((WPB + 1) * kWave);
    const Table &t = a.tab[0];
    const u64x4 pointers = {word_of(a.keys), word_of(t.K), word_of(t.epoch), word_of(a.n_dev)};
    const u32x4 sizes = {a.B, a.kpw | a.deal << 16, a.tiles_per_table, a.n_tiles};
    const u32x2 sets = {t.S, t.smask};
    if constexpr (WPB <= 8 || W <= 16) {           // query_shape gives no more than 8 workers to wider sets
#define HPS_QUERY(full) \
    hipLaunchKernelGGL((query_kernel<W, kWave, U, WPB, kCoherent, kD, full>), grid, block, 0, st, pointers, sizes, sets, a)
        if (full) HPS_QUERY(true);
        else      HPS_QUERY(false);
#undef HPS_QUERY
    }
}

template <int W, int WPB>
void launch_query_dedup(const QueryArgs &a, hipStream_t st) {
    const uint32_t grid = a.n_tiles < (1u << 20) ? a.n_tiles : (1u << 20);
    hipLaunchKernelGGL((query_dedup_kernel<W, (WPB == 8 ? 4 : 8), WPB>), dim3(grid), dim3((WPB + 1) * kWave), 0, st, a);
}

template <int W>
hps_status_t launch_query_w(const QueryArgs &a, QueryShape q, bool coherent, bool dedup, bool full, hipStream_t st) {
    const int id = q.u * 100 + q.wpb;
    const bool d128 = a.g.d == 128;
    if (dedup) {
        if (q.wpb == 4) launch_query_dedup<W, 4>(a, st);
        else launch_query_dedup<W, 8>(a, st);
    } else if (coherent) {
        switch (d128 ? 10000 + id : id) {
            case 10404: launch_query_kernel<W, 4, 4, true, 128>(a, full, st); break;
            case 10804: launch_query_kernel<W, 8, 4, true, 128>(a, full, st); break;
            case 11604: launch_query_kernel<W, 16, 4, true, 128>(a, full, st); break;
            case 11605: launch_query_kernel<W, 16, 5, true, 128>(a, full, st); break;
            case 11607: launch_query_kernel<W, 16, 7, true, 128>(a, full, st); break;
            case 13207: launch_query_kernel<W, 32, 7, true, 128>(a, full, st); break;
            case 804: launch_query_kernel<W, 8, 4, true, 0>(a, full, st); break;
            case 1604: launch_query_kernel<W, 16, 4, true, 0>(a, full, st); break;
            case 3204: launch_query_kernel<W, 32, 4, true, 0>(a, full, st); break;
            case 805: launch_query_kernel<W, 8, 5, true, 0>(a, full, st); break;
            case 1605: launch_query_kernel<W, 16, 5, true, 0>(a, full, st); break;
            case 3205: launch_query_kernel<W, 32, 5, true, 0>(a, full, st); break;
            case 807: launch_query_kernel<W, 8, 7, true, 0>(a, full, st); break;
            case 1607: launch_query_kernel<W, 16, 7, true, 0>(a, full, st); break;
            case 3207: launch_query_kernel<W, 32, 7, true, 0>(a, full, st); break;
            case 811: launch_query_kernel<W, 8, 11, true, 0>(a, full, st); break;
            case 1611: launch_query_kernel<W, 16, 11, true, 0>(a, full, st); break;
            default: return fail(HPS_ERR_INVALID_ARG, "query shape not compiled in");
        }
    } else {
        switch (d128 ? 10000 + id : id) {
            case 10404: launch_query_kernel<W, 4, 4, false, 128>(a, full, st); break;
            case 10804: launch_query_kernel<W, 8, 4, false, 128>(a, full, st); break;
            case 11604: launch_query_kernel<W, 16, 4, false, 128>(a, full, st); break;
            case 11605: launch_query_kernel<W, 16, 5, false, 128>(a, full, st); break;
            case 11607: launch_query_kernel<W, 16, 7, false, 128>(a, full, st); break;
            case 13207: launch_query_kernel<W, 32, 7, false, 128>(a, full, st); break;
            case 13208: launch_query_kernel<W, 32, 8, false, 128>(a, full, st); break;
            case 804: launch_query_kernel<W, 8, 4, false, 0>(a, full, st); break;
            case 1604: launch_query_kernel<W, 16, 4, false, 0>(a, full, st); break;
            case 3204: launch_query_kernel<W, 32, 4, false, 0>(a, full, st); break;
            case 805: launch_query_kernel<W, 8, 5, false, 0>(a, full, st); break;
            case 1605: launch_query_kernel<W, 16, 5, false, 0>(a, full, st); break;
            case 3205: launch_query_kernel<W, 32, 5, false, 0>(a, full, st); break;
            case 807: launch_query_kernel<W, 8, 7, false, 0>(a, full, st); break;
            case 1607: launch_query_kernel<W, 16, 7, false, 0>(a, full, st); break;
            case 3207: launch_query_kernel<W, 32, 7, false, 0>(a, full, st); break;
            case 811: launch_query_kernel<W, 8, 11, false, 0>(a, full, st); break;
            case 1611: launch_query_kernel<W, 16, 11, false, 0>(a, full, st); break;
            case 815: launch_query_kernel<W, 8, 15, false, 0>(a, full, st); break;
            default: return fail(HPS_ERR_INVALID_ARG, "query shape not compiled in");
        }
    }
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t launch_query(uint32_t W, const QueryArgs &a, QueryShape q, bool coherent, bool dedup,
                          bool full, hipStream_t st) {
    switch (W) {
        case 1:  return launch_query_w<1>(a, q, coherent, dedup, full, st);
        case 2:  return launch_query_w<2>(a, q, coherent, dedup, full, st);
        case 4:  return launch_query_w<4>(a, q, coherent, dedup, full, st);
        case 8:  return launch_query_w<8>(a, q, coherent, dedup, full, st);
        case 16: return launch_query_w<16>(a, q, coherent, dedup, full, st);
        case 32: return launch_query_w<32>(a, q, coherent, dedup, full, st);
        case 64: return launch_query_w<64>(a, q, coherent, dedup, full, st);
        default: return fail(HPS_ERR_INVALID_ARG, "unsupported ways");
    }
}

template <bool kInsert>
hps_status_t launch_write(hps_cache *c, const int64_t *keys, const float *vals, size_t n,
                          const uint32_t *n_dev, hipStream_t st) {
    const Table t = table_of(c);
    const WriteArgs a{vals, t.V, t.T, t.gdev, t.flags, make_geom(c->d)};
    const u64x4 pointers = {word_of(keys), word_of(n_dev), word_of(t.K), word_of(t.sc)};
    const u32x4 sizes = {(uint32_t)n, t.S, t.smask, 0u};
    // Insert: 16 keys per wave, 8 while 4,096 waves (four per SIMD) hold the batch that way: 8,192 rows 12.1 -> 9.7 us,
    // 32,768 rows 16.8 -> 15.7; with 8 throughout the 425,984-key streaming step takes 166 instead of 149 us.
    // (32 and 64 are 3-45 % slower than 16 from 1 K to 1 M keys.)
    // Update: 64 keys per wave, 16 for batches below 32,768 keys: 8,192 rows 14.1 us (64s: 23, 8s: 13.4, but a dump's
    // keys come eight to a set, and 8s split sets between waves: dump + update + query of 28,000 rows of 256
    // bytes 28.6 instead of 26.0); on a 40 GB refresh 64s are 9-55 % faster.
    // Up to 49,152 keys 16 where the rows are long enough to outweigh that in a dump's order the waves wait for each other's sets.  16s / 64s,
    // random order and a dump's: 40,000 rows of 512 bytes, 8 ways 25.1 / 29.5 and 15.2 / 17.2, 256 bytes 20.2 / 24.3 and 11.8 / 11.4, but 128 bytes
    // 19.1 / 20.9 and 11.0 / 9.7; 33,000 rows, 16 ways, 256 bytes 25 / 33 and 12.1 / 13.7, 128 bytes 24 / 26 and 12.3 / 11.0; 32 ways, 512 bytes 46 / 60 and
    // 20 / 22, 256 bytes 42 / 55 and 19.4 / 16.8; 64 ways, 512 bytes 90 / 132 and 44 / 29.  49,152 rows of 512 bytes, 8 ways 28.2 / 31.1 and 17.2 / 18.1,
    // 60,000 33.6 / 35.2 and 20.2 / 18.7.
    const uint32_t least = c->W <= 4 ? 16 * c->W : c->W <= 16 ? 64u : c->W <= 32 ? 128u : ~0u;
    const uint32_t kpw = kInsert ? (n <= 32768 ? 8u : 16u) : (n < 32768 || (n <= 49152 && c->d >= least) ? 16u : (uint32_t)kWave);
    const uint64_t tiles = (n + kpw - 1) / kpw;
    const uint64_t blocks = (tiles + kWavesPerWg - 1) / kWavesPerWg;
    const dim3 grid((uint32_t)(blocks < kWriteGridX ? blocks : kWriteGridX), (uint32_t)((blocks + kWriteGridX - 1) / kWriteGridX)), block(kBlock);
    const bool lng = c->d > 256;               // rows of more than one wave load
    switch (c->W) {
#define HPS_LAUNCH(...) hipLaunchKernelGGL((__VA_ARGS__), grid, block, 0, st, pointers, sizes, word_of(t.epoch), a)
#define HPS_INSERT(w, lru)                                                                  \
    do {                                                                                    \
        if (kpw == 8 && lng) HPS_LAUNCH(insert_kernel<w, 8, true, lru>);                    \
        else if (kpw == 8) HPS_LAUNCH(insert_kernel<w, 8, false, lru>);                     \
        else if (lng) HPS_LAUNCH(insert_kernel<w, 16, true, lru>);                          \
        else HPS_LAUNCH(insert_kernel<w, 16, false, lru>);                                  \
    } while (0)
#define HPS_CASE(w)                                                                         \
    case w:                                                                                 \
        if (kInsert) {                                                                      \
            if (t.T) HPS_INSERT(w, true);                                               \
            else HPS_INSERT(w, false);                                                      \
        } else if (kpw == 16) {                                                             \
            if (lng) HPS_LAUNCH(update_kernel<w, 16, true>);                                \
            else HPS_LAUNCH(update_kernel<w, 16, false>);                                   \
        } else {                                                                            \
            if (lng) HPS_LAUNCH(update_kernel<w, 64, true>);                                \
            else HPS_LAUNCH(update_kernel<w, 64, false>);                                   \
        }                                                                                   \
        break;
        HPS_CASE(1) HPS_CASE(2) HPS_CASE(4) HPS_CASE(8) HPS_CASE(16) HPS_CASE(32) HPS_CASE(64)
#undef HPS_CASE
#undef HPS_INSERT
#undef HPS_LAUNCH
        default: return fail(HPS_ERR_INVALID_ARG, "unsupported ways");
    }
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t write_call(hps_cache *c, const int64_t *keys, const float *vals, size_t n,
                        const uint32_t *n_dev, void *stream, bool insert) {
    if (hps_status_t s = check_handle(c)) return s;
    if (n == 0) return HPS_OK;
    if (n >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n must be < 2^32");
    if (!keys || !vals) return fail(HPS_ERR_INVALID_ARG, "keys/vals must not be NULL when n > 0");
    if (!aligned(keys, 8) || !aligned(vals, 16) || !aligned(n_dev, 4))
        return fail(HPS_ERR_INVALID_ARG, "keys must be 8-byte and vals 16-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(stream);
    return insert ? launch_write<true>(c, keys, vals, n, n_dev, st)
                  : launch_write<false>(c, keys, vals, n, n_dev, st);
}

}  // namespace

// ------------------------------------------------------------------ C ABI

hipError_t hps_launch_expand_rows(const float *rows, const uint32_t *inverse, uint32_t n, uint32_t dim, float *out,
                                  uint32_t cus, hipStream_t st) {
    // 8 waves per work-group, keys per wave for full rounds of them, a wave's rows in one group of wave loads.  A launch has fewer than 2^32
    // work-items, and there is one for each position or more: at most 2^30 positions go in one (a quarter of what a call may have).
    constexpr uint32_t kWpb = 8, kMost = 1u << 30;
    const RowGeom g = make_geom(dim);
    for (uint32_t done = 0; done < n;) {
        const uint32_t m = n - done < kMost ? n - done : kMost;
        const uint64_t rounds = ((uint64_t)m + kWpb * kWave * cus - 1) / (kWpb * kWave * cus);
        uint64_t kpw = ((uint64_t)m + kWpb * cus * rounds - 1) / (kWpb * cus * rounds);
        // Fewer rows per wave than the floor where they are long and waves are free: 100 rows of 16 KiB, eight to a wave, took
        // 20.4 us, two to a wave 6.7; 3,000 of them 24.5 and 14.3.
        const uint64_t floor_k = m < 4096 ? kMinKeysPerWave : 16, fit = (8192 + dim / 2) / dim;   // about 32 KiB
        const uint64_t least = fit < 1 ? 1 : fit < floor_k ? fit : floor_k;
        if (kpw < least) kpw = least;
        if (kpw > most_rows(dim)) kpw = most_rows(dim);
        const uint32_t blocks = (uint32_t)(((uint64_t)m + kWpb * kpw - 1) / (kWpb * kpw));
        const uint64_t bytes = kpw * dim * 4;
        const uint32_t *const inv = inverse + done;
        float *const to = out + (uint64_t)done * dim;
#define HPS_EXPAND(U, D) \
    hipLaunchKernelGGL((expand_rows_kernel<U, kWpb, D>), dim3(blocks), dim3(kWpb * kWave), 0, st, rows, inv, m, (uint32_t)kpw, g, to)
        if (dim == 128) {
            if (bytes <= 13312) HPS_EXPAND(13, 128);
            else if (bytes <= 26624) HPS_EXPAND(26, 128);
            else HPS_EXPAND(32, 128);
        } else {
            if (bytes <= 8192) HPS_EXPAND(8, 0);
            else if (bytes <= 16384) HPS_EXPAND(16, 0);
            else HPS_EXPAND(32, 0);
        }
#undef HPS_EXPAND
        done += m;
    }
    return hipGetLastError();
}

extern "C" {

const char *hps_last_error(void) { return g_err.c_str(); }

hps_status_t hps_cache_create(size_t capacity, uint32_t ways, uint32_t dim, hps_cache_t **out_handle) {
    return hps_cache_create_policy(capacity, ways, dim, HPS_POLICY_VICTIM_COUNTER, out_handle);
}

hps_status_t hps_cache_create_policy(size_t capacity, uint32_t ways, uint32_t dim, int policy,
                                     hps_cache_t **out_handle) {
    if (!out_handle) return fail(HPS_ERR_INVALID_ARG, "out_handle is NULL");
    *out_handle = nullptr;
    if (policy != HPS_POLICY_VICTIM_COUNTER && policy != HPS_POLICY_LRU)
        return fail(HPS_ERR_INVALID_ARG, "unknown replacement policy");
    if (ways == 0 || ways > 64 || (ways & (ways - 1)) != 0)
        return fail(HPS_ERR_INVALID_ARG, "ways must be a power of two in [1, 64]");
    if (capacity == 0 || capacity % ways != 0)
        return fail(HPS_ERR_INVALID_ARG, "capacity must be a non-zero multiple of ways");
    if (capacity / ways >= (1ull << 31))
        return fail(HPS_ERR_INVALID_ARG, "capacity / ways must be < 2^31");
    if (dim == 0 || dim % 4 != 0) return fail(HPS_ERR_INVALID_ARG, "dim must be a non-zero multiple of 4");

    hps_cache *c = new (std::nothrow) hps_cache();
    if (!c) return fail(HPS_ERR_OOM, "host allocation failed");
    c->magic = kMagic;
    c->S = capacity / ways;
    c->W = ways;
    c->d = dim;
    c->K = nullptr; c->V = nullptr; c->sc = nullptr; c->ring = nullptr; c->T = nullptr; c->flags = nullptr;
    c->epoch = nullptr; c->word_half = 0;
    c->policy = policy;
    c->concurrent_writers.store(dim <= kMaxCheckedDim ? 1 : 0);
    c->query_dedup.store(0);

    hipError_t e = hipGetDevice(&c->device);
    c->n_cus = 256;
    if (e == hipSuccess) e = hipDeviceGetAttribute(&c->n_cus, hipDeviceAttributeMultiprocessorCount, c->device);
    if (e == hipSuccess && c->n_cus <= 0) c->n_cus = 256;
    if (e == hipSuccess) e = hipMalloc(&c->K, capacity * sizeof(int64_t));
    if (e == hipSuccess) e = hipMalloc(&c->V, capacity * (size_t)dim * sizeof(float));
    if (e == hipSuccess) e = hipMalloc(&c->sc, c->S * 2 * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMalloc(&c->ring, 2 * kRing * sizeof(uint64_t));
    if (e == hipSuccess) e = hipMalloc(&c->flags, 2 * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMemsetAsync(c->flags, 0, 2 * sizeof(uint32_t), 0);
    constexpr size_t kEpochBytes = kEpochs * kEpochStride * sizeof(uint32_t);
    if (e == hipSuccess) e = hipMalloc(&c->epoch, kEpochBytes);
    if (e == hipSuccess) e = hipMemsetAsync(c->epoch, 0, kEpochBytes, 0);
    if (e == hipSuccess && policy == HPS_POLICY_LRU) {
        e = hipMalloc(&c->T, capacity * sizeof(uint32_t));
        if (e == hipSuccess) e = hipMemsetAsync(c->T, 0, capacity * sizeof(uint32_t), 0);
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(fill_keys_kernel, dim3(4096), dim3(256), 0, 0, c->K, (uint64_t)capacity, kEmpty);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemsetAsync(c->V, 0, capacity * (size_t)dim * sizeof(float), 0);
    if (e == hipSuccess) e = hipMemsetAsync(c->sc, 0, c->S * 2 * sizeof(uint32_t), 0);
    if (e == hipSuccess) e = hipMemsetAsync(c->ring, 0, 2 * kRing * sizeof(uint64_t), 0);
    if (e == hipSuccess) e = hipStreamSynchronize(0);
    if (e != hipSuccess) {
        const hps_status_t code = e == hipErrorOutOfMemory ? HPS_ERR_OOM : HPS_ERR_DEVICE;
        std::string msg = std::string("hps_cache_create: ") + hipGetErrorString(e);
        (void)hipGetLastError();
        if (c->K) (void)hipFree(c->K);
        if (c->V) (void)hipFree(c->V);
        if (c->sc) (void)hipFree(c->sc);
        if (c->ring) (void)hipFree(c->ring);
        if (c->T) (void)hipFree(c->T);
        if (c->flags) (void)hipFree(c->flags);
        if (c->epoch) (void)hipFree(c->epoch);
        delete c;
        return fail(code, msg);
    }
    *out_handle = c;
    return HPS_OK;
}

hps_status_t hps_cache_destroy(hps_cache_t *c) {
    if (!c || c->magic != kMagic) return fail(HPS_ERR_INVALID_ARG, "invalid cache handle");
    c->magic = 0;
    hipError_t e = hipSuccess, e2;
    if ((e2 = hipFree(c->K)) != hipSuccess) e = e2;
    if ((e2 = hipFree(c->V)) != hipSuccess) e = e2;
    if ((e2 = hipFree(c->sc)) != hipSuccess) e = e2;
    if ((e2 = hipFree(c->ring)) != hipSuccess) e = e2;
    if (c->T && (e2 = hipFree(c->T)) != hipSuccess) e = e2;
    if ((e2 = hipFree(c->flags)) != hipSuccess) e = e2;
    if ((e2 = hipFree(c->epoch)) != hipSuccess) e = e2;
    delete c;
    if (e != hipSuccess) return fail(HPS_ERR_DEVICE, std::string("hipFree: ") + hipGetErrorString(e));
    return HPS_OK;
}

hps_status_t hps_cache_info(const hps_cache_t *c, uint64_t *num_sets, uint32_t *ways, uint32_t *dim) {
    if (!c || c->magic != kMagic) return fail(HPS_ERR_INVALID_ARG, "invalid cache handle");
    if (num_sets) *num_sets = c->S;
    if (ways) *ways = c->W;
    if (dim) *dim = c->d;
    return HPS_OK;
}

hps_status_t hps_cache_set_concurrent_writers(hps_cache_t *c, int enabled) {
    if (!c || c->magic != kMagic) return fail(HPS_ERR_INVALID_ARG, "invalid cache handle");
    if (enabled && c->d > kMaxCheckedDim)
        return fail(HPS_ERR_INVALID_ARG, "queries overlapping writers are supported for dim <= " +
                                             std::to_string(kMaxCheckedDim) + " (4 KiB rows)");
    c->concurrent_writers.store(enabled ? 1 : 0);
    return HPS_OK;
}

hps_status_t hps_cache_flags(hps_cache_t *c, uint32_t *flags, int clear) {
    if (hps_status_t s = check_handle(c)) return s;
    if (!flags) return fail(HPS_ERR_INVALID_ARG, "flags is NULL");
    HIP_TRY(hipMemcpy(flags, c->flags, sizeof(uint32_t), hipMemcpyDeviceToHost));
    if (clear) HIP_TRY(hipMemset(c->flags, 0, sizeof(uint32_t)));
    return HPS_OK;
}

hps_status_t hps_cache_debug_set_seq(hps_cache_t *c, uint64_t set, uint32_t value) {
    if (hps_status_t s = check_handle(c)) return s;
    if (set >= c->S) return fail(HPS_ERR_INVALID_ARG, "set index out of range");
    hipLaunchKernelGGL(set_seq_kernel, dim3(1), dim3(1), 0, 0, c->sc + 2 * set, value, c->epoch);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(0));
    return HPS_OK;
}

hps_status_t hps_cache_debug_writers(hps_cache_t *c, uint32_t *started, uint32_t *finished) {
    if (hps_status_t s = check_handle(c)) return s;
    if (!started || !finished) return fail(HPS_ERR_INVALID_ARG, "started and finished must not be NULL");
    uint32_t pairs[kEpochs * kEpochStride];
    HIP_TRY(hipMemcpy(pairs, c->epoch, sizeof(pairs), hipMemcpyDeviceToHost));
    *started = *finished = 0;
    for (uint32_t i = 0; i < kEpochs; ++i) {
        *started += pairs[i * kEpochStride];
        *finished += pairs[i * kEpochStride + 1];
    }
    return HPS_OK;
}

hps_status_t hps_cache_set_query_dedup(hps_cache_t *c, int enabled) {
    if (!c || c->magic != kMagic) return fail(HPS_ERR_INVALID_ARG, "invalid cache handle");
    c->query_dedup.store(enabled ? 1 : 0);
    return HPS_OK;
}

static hps_status_t query_call(hps_cache_t *const *caches, uint32_t n_tables, const int64_t *keys,
                               size_t batch, const uint32_t *n_dev, float *out, uint32_t *miss_idx,
                               int64_t *miss_keys, uint32_t *n_miss, void *stream) {
    if (!caches || n_tables == 0 || n_tables > HPS_MAX_TABLES)
        return fail(HPS_ERR_INVALID_ARG, "n_tables must be in [1, HPS_MAX_TABLES]");
    for (uint32_t t = 0; t < n_tables; ++t) {
        if (hps_status_t s = check_handle(caches[t])) return s;
        if (caches[t]->d != caches[0]->d || caches[t]->W != caches[0]->W)
            return fail(HPS_ERR_INVALID_ARG, "all tables of one call must share dim and ways");
    }
    if (!n_miss || !aligned(n_miss, 4)) return fail(HPS_ERR_INVALID_ARG, "n_miss must be a 4-byte aligned device pointer");
    const uint64_t total = (uint64_t)n_tables * batch;
    if (total >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n_tables * batch must be < 2^32");
    if (total > 0) {
        if (!keys || !out || !miss_idx || !miss_keys)
            return fail(HPS_ERR_INVALID_ARG, "keys/out/miss_idx/miss_keys must not be NULL when n > 0");
        if (!aligned(keys, 8) || !aligned(miss_keys, 8) || !aligned(out, 16) || !aligned(miss_idx, 4))
            return fail(HPS_ERR_INVALID_ARG, "misaligned buffer (keys 8, out 16, miss_idx 4 bytes)");
    }
    QueryArgs a;
    std::memset(&a, 0, sizeof(a));
    for (uint32_t t = 0; t < n_tables; ++t) a.tab[t] = table_of(caches[t]);
    a.n_tables = n_tables;
    a.keys = keys;
    a.out = out;
    a.miss_idx = miss_idx;
    a.miss_keys = miss_keys;
    a.n_miss = n_miss;
    a.slot = counter_word(caches[0], stream);
    a.B = (uint32_t)batch;
    a.n_dev = n_dev;
    bool coherent = false;                      // any table that may see concurrent writers makes the call careful
    for (uint32_t t = 0; t < n_tables; ++t) coherent = coherent || caches[t]->concurrent_writers.load() != 0;
    const bool dedup = !coherent && caches[0]->query_dedup.load() != 0;
    const QueryShape shape = query_shape(n_tables, batch, caches[0]->d, (uint64_t)caches[0]->n_cus, coherent, dedup, caches[0]->W, n_dev != nullptr);
    const uint32_t kpw = shape.kpw;
    a.kpw = kpw;
    a.deal = shape.deal;
    const uint32_t tile = kpw * (uint32_t)shape.wpb;
    a.tiles_per_table = (uint32_t)((batch + tile - 1) / tile);
    if (a.tiles_per_table == 0) a.tiles_per_table = 1;          // an empty batch still publishes n_miss = 0
    a.n_tiles = a.tiles_per_table * n_tables;
    a.g = make_geom(caches[0]->d);
    bool full = n_dev != nullptr;               // a device-side length or any LRU table (Alg. 2 stamps) selects the full kernels
    for (uint32_t t = 0; t < n_tables; ++t) full = full || a.tab[t].T != nullptr;
    return launch_query(caches[0]->W, a, shape, coherent, dedup, full, static_cast<hipStream_t>(stream));
}

hps_status_t hps_cache_query_multi(hps_cache_t *const *caches, uint32_t n_tables, const int64_t *keys,
                                   size_t batch, float *out, uint32_t *miss_idx, int64_t *miss_keys,
                                   uint32_t *n_miss, void *stream) {
    return query_call(caches, n_tables, keys, batch, nullptr, out, miss_idx, miss_keys, n_miss, stream);
}

hps_status_t hps_cache_query(hps_cache_t *c, const int64_t *keys, size_t n, float *out,
                             uint32_t *miss_idx, int64_t *miss_keys, uint32_t *n_miss, void *stream) {
    if (n >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n must be < 2^32");
    hps_cache_t *one[1] = {c};
    return query_call(one, 1, keys, n, nullptr, out, miss_idx, miss_keys, n_miss, stream);
}

hps_status_t hps_cache_query_dn(hps_cache_t *c, const int64_t *keys, size_t n_max, const uint32_t *n_dev,
                                float *out, uint32_t *miss_idx, int64_t *miss_keys, uint32_t *n_miss,
                                void *stream) {
    if (n_max >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n_max must be < 2^32");
    if (!n_dev || !aligned(n_dev, 4)) return fail(HPS_ERR_INVALID_ARG, "n_dev must be a 4-byte aligned device pointer");
    hps_cache_t *one[1] = {c};
    return query_call(one, 1, keys, n_max, n_dev, out, miss_idx, miss_keys, n_miss, stream);
}

hps_status_t hps_cache_insert(hps_cache_t *c, const int64_t *keys, const float *vals, size_t n, void *stream) {
    return write_call(c, keys, vals, n, nullptr, stream, true);
}
hps_status_t hps_cache_update(hps_cache_t *c, const int64_t *keys, const float *vals, size_t n, void *stream) {
    return write_call(c, keys, vals, n, nullptr, stream, false);
}
hps_status_t hps_cache_insert_dn(hps_cache_t *c, const int64_t *keys, const float *vals, size_t n_max,
                                 const uint32_t *n_dev, void *stream) {
    if (!n_dev) return fail(HPS_ERR_INVALID_ARG, "n_dev is NULL");
    return write_call(c, keys, vals, n_max, n_dev, stream, true);
}
hps_status_t hps_cache_update_dn(hps_cache_t *c, const int64_t *keys, const float *vals, size_t n_max,
                                 const uint32_t *n_dev, void *stream) {
    if (!n_dev) return fail(HPS_ERR_INVALID_ARG, "n_dev is NULL");
    return write_call(c, keys, vals, n_max, n_dev, stream, false);
}

hps_status_t hps_cache_export(hps_cache_t *c, int64_t *keys, uint32_t *ctr, float *vals, void *stream) {
    if (hps_status_t s = check_handle(c)) return s;
    if (!keys || !ctr) return fail(HPS_ERR_INVALID_ARG, "keys and ctr must not be NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t slots = c->S * c->W;
    HIP_TRY(hipMemcpyAsync(keys, c->K, slots * sizeof(int64_t), hipMemcpyDeviceToDevice, st));
    hipLaunchKernelGGL(counters_out_kernel, dim3(1024), dim3(256), 0, st, c->sc, (uint64_t)c->S, ctr);
    HIP_TRY(hipGetLastError());
    if (vals)
        HIP_TRY(hipMemcpyAsync(vals, c->V, slots * c->d * sizeof(float), hipMemcpyDeviceToDevice, st));
    return HPS_OK;
}

hps_status_t hps_cache_import(hps_cache_t *c, const int64_t *keys, const uint32_t *ctr, const float *vals,
                              void *stream) {
    if (hps_status_t s = check_handle(c)) return s;
    if (!keys || !ctr) return fail(HPS_ERR_INVALID_ARG, "keys and ctr must not be NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t slots = c->S * c->W;
    HIP_TRY(hipMemcpyAsync(c->K, keys, slots * sizeof(int64_t), hipMemcpyDeviceToDevice, st));
    if (vals)
        HIP_TRY(hipMemcpyAsync(c->V, vals, slots * c->d * sizeof(float), hipMemcpyDeviceToDevice, st));
    hipLaunchKernelGGL(counters_in_kernel, dim3(1024), dim3(256), 0, st, c->sc, (uint64_t)c->S, ctr, c->epoch);
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t hps_cache_export_lru(hps_cache_t *c, uint32_t *stamps, uint32_t *g, void *stream) {
    if (hps_status_t s = check_handle(c)) return s;
    if (c->policy != HPS_POLICY_LRU) return fail(HPS_ERR_INVALID_ARG, "the cache was not created with the LRU policy");
    if (!stamps || !g) return fail(HPS_ERR_INVALID_ARG, "stamps and g must not be NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    HIP_TRY(hipMemcpyAsync(stamps, c->T, c->S * c->W * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
    HIP_TRY(hipMemcpyAsync(g, c->flags + 1, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));                   // *g is a host word: it is valid on return
    return HPS_OK;
}

hps_status_t hps_cache_import_lru(hps_cache_t *c, const uint32_t *stamps, uint32_t g, void *stream) {
    if (hps_status_t s = check_handle(c)) return s;
    if (c->policy != HPS_POLICY_LRU) return fail(HPS_ERR_INVALID_ARG, "the cache was not created with the LRU policy");
    if (!stamps) return fail(HPS_ERR_INVALID_ARG, "stamps must not be NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    HIP_TRY(hipMemcpyAsync(c->T, stamps, c->S * c->W * sizeof(uint32_t), hipMemcpyDeviceToDevice, st));
    hipLaunchKernelGGL(set_u32_kernel, dim3(1), dim3(1), 0, st, c->flags + 1, g);
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t hps_cache_dump(hps_cache_t *c, size_t first_slot, size_t n_slots, int64_t *keys_out,
                            uint32_t *n_out, void *stream) {
    if (hps_status_t s = check_handle(c)) return s;
    const size_t slots = c->S * c->W;
    if (first_slot > slots || n_slots > slots - first_slot)
        return fail(HPS_ERR_INVALID_ARG, "slot range exceeds the cache");
    if (n_slots >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n_slots must be < 2^32 per call");
    if (!n_out || (n_slots > 0 && !keys_out)) return fail(HPS_ERR_INVALID_ARG, "output pointer is NULL");
    if (!aligned(keys_out, 8) || !aligned(n_out, 4)) return fail(HPS_ERR_INVALID_ARG, "misaligned output buffer");
    constexpr int kDumpKpt = 32;                       // 8192 slots per tile (16 and 64 dump 15-20 % slower)
    uint32_t n_tiles = (uint32_t)((n_slots + kBlock * kDumpKpt - 1) / (kBlock * kDumpKpt));
    if (n_tiles == 0) n_tiles = 1;
    const uint32_t grid = n_tiles < (1u << 20) ? n_tiles : (1u << 20);
    hipLaunchKernelGGL((dump_kernel<kDumpKpt>), dim3(grid), dim3(kBlock), 0, static_cast<hipStream_t>(stream), c->K,
                       (uint64_t)first_slot, (uint64_t)n_slots, keys_out, n_out, counter_word(c, stream), n_tiles);
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t hps_membench_gather(const float *rows, const uint32_t *slot_of, size_t n, uint32_t dim, float *out,
                                 void *stream) {
    if (dim == 0 || dim % 4 != 0) return fail(HPS_ERR_INVALID_ARG, "dim must be a non-zero multiple of 4");
    if (n == 0) return HPS_OK;
    if (n >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n must be < 2^32");
    if (!rows || !slot_of || !out) return fail(HPS_ERR_INVALID_ARG, "rows, slot_of and out must not be NULL");
    if (!aligned(rows, 16) || !aligned(out, 16) || !aligned(slot_of, 4)) return fail(HPS_ERR_INVALID_ARG, "misaligned buffer");
    int dev = 0, cus = 256;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (cus <= 0) cus = 256;
    // the worker waves and the keys per wave of a large query (query_shape)
    constexpr int kWpb = 7;
    const uint64_t kpw = query_shape(1, n, dim, (uint64_t)cus, false, false).kpw;
    const uint64_t tile = kpw * kWpb;
    const uint64_t blocks = (n + tile - 1) / tile;
    if (blocks >= (1ull << 31)) return fail(HPS_ERR_INVALID_ARG, "n too large");
    if (dim == 128)
        hipLaunchKernelGGL((membench_gather_kernel<32, kWpb, 128>), dim3((uint32_t)blocks), dim3(kWpb * kWave), 0,
                           static_cast<hipStream_t>(stream), rows, slot_of, (uint32_t)n, (uint32_t)kpw, make_geom(dim), out);
    else
        hipLaunchKernelGGL((membench_gather_kernel<32, kWpb, 0>), dim3((uint32_t)blocks), dim3(kWpb * kWave), 0,
                           static_cast<hipStream_t>(stream), rows, slot_of, (uint32_t)n, (uint32_t)kpw, make_geom(dim), out);
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t hps_membench_gather_half(const float *rows, const uint32_t *slot_of, size_t n, float *out,
                                      int reads, void *stream) {
    if (n == 0) return HPS_OK;
    if (!rows || !slot_of || !out) return fail(HPS_ERR_INVALID_ARG, "null pointer");
    if (n >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n must be < 2^32");
    if (!aligned(rows, 16) || !aligned(out, 16)) return fail(HPS_ERR_INVALID_ARG, "rows and out must be 16-byte aligned");
    int dev = 0, cus = 256;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (cus <= 0) cus = 256;
    constexpr int kWpb = 7;                     // the shape hps_membench_gather uses
    const uint64_t kpw = query_shape(1, n, 128, (uint64_t)cus, false, false).kpw;
    const uint64_t tile = kpw * kWpb;
    const uint64_t blocks = (n + tile - 1) / tile;
    if (blocks >= (1ull << 31)) return fail(HPS_ERR_INVALID_ARG, "n too large");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (reads)
        hipLaunchKernelGGL((membench_half_kernel<32, kWpb, true>), dim3((uint32_t)blocks), dim3(kWpb * kWave), 0, st,
                           rows, slot_of, (uint32_t)n, (uint32_t)kpw, out);
    else
        hipLaunchKernelGGL((membench_half_kernel<32, kWpb, false>), dim3((uint32_t)blocks), dim3(kWpb * kWave), 0, st,
                           rows, slot_of, (uint32_t)n, (uint32_t)kpw, out);
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t hps_membench_copy(const void *src, void *dst, size_t bytes, int nontemporal, void *stream) {
    if (bytes == 0) return HPS_OK;
    if (!src || !dst || bytes % 16 != 0 || !aligned(src, 16) || !aligned(dst, 16))
        return fail(HPS_ERR_INVALID_ARG, "src and dst must be 16-byte aligned and bytes a multiple of 16");
    const uint64_t n16 = bytes / 16;
    uint64_t blocks = (n16 + (uint64_t)kBlock * 8 - 1) / ((uint64_t)kBlock * 8);
    if (blocks > 16384) blocks = 16384;
    if (blocks == 0) blocks = 1;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (nontemporal)
        hipLaunchKernelGGL((membench_copy_kernel<8, true>), dim3((uint32_t)blocks), dim3(kBlock), 0, st,
                           static_cast<const f32x4 *>(src), static_cast<f32x4 *>(dst), n16);
    else
        hipLaunchKernelGGL((membench_copy_kernel<8, false>), dim3((uint32_t)blocks), dim3(kBlock), 0, st,
                           static_cast<const f32x4 *>(src), static_cast<f32x4 *>(dst), n16);
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t hps_backing_fetch(const int64_t *keys, size_t n, const uint32_t *n_dev, uint32_t dim,
                               uint32_t version, float *rows, const uint32_t *scatter_idx,
                               float *scatter_out, void *stream) {
    if (dim == 0 || dim % 4 != 0) return fail(HPS_ERR_INVALID_ARG, "dim must be a non-zero multiple of 4");
    if (n == 0) return HPS_OK;
    if (n >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n must be < 2^32");
    if (!keys || (!rows && !scatter_idx)) return fail(HPS_ERR_INVALID_ARG, "keys and one output are required");
    if (scatter_idx && !scatter_out) return fail(HPS_ERR_INVALID_ARG, "scatter_out is NULL");
    if (!aligned(keys, 8) || !aligned(rows, 16) || !aligned(scatter_out, 16) || !aligned(scatter_idx, 4))
        return fail(HPS_ERR_INVALID_ARG, "misaligned buffer");
    const RowGeom g = make_geom(dim);
    const uint64_t per_block = (uint64_t)kWavesPerWg * ((uint32_t)kWave >> g.lprShift);
    uint64_t blocks = (n + per_block - 1) / per_block * g.passes;
    if (blocks > kBackingWaves / kWavesPerWg) blocks = kBackingWaves / kWavesPerWg;
    if (rows && scatter_idx)
        hipLaunchKernelGGL((backing_kernel<true>), dim3((uint32_t)blocks), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                           keys, (uint32_t)n, n_dev, version, g, rows, scatter_idx, scatter_out);
    else
        hipLaunchKernelGGL((backing_kernel<false>), dim3((uint32_t)blocks), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                           keys, (uint32_t)n, n_dev, version, g, rows, scatter_idx, scatter_out);
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

}  // extern "C"

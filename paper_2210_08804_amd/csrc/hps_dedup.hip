// Deduplication operator Q* = dedup(Q) of the paper's Sec. 2.2 and the row expansion that
// follows the lookup of Q*, for gfx950.
//
// dedup is a hash join of the batch with itself in one launch over an open-addressing table (one
// 8-byte key word and one 4-byte number per slot, 2n..16n slots).  A session has two tables: a call works
// on the clean one and wipes the part of the other one that the previous call used, so no call
// waits for a clear.  A work-group takes 1024 (or 512) keys and
//   elects one lane per distinct key of the tile in an LDS table (so a hot key reaches the global table
//   once per tile, not once per occurrence),
//   lets the elected lanes claim a slot of the global table with a 64-bit compare-and-swap,
//   numbers the lanes whose swap succeeded (one global counter atomic per tile) and writes their key to
//   unique_keys and their number beside the slot,
//   reads the numbers of the keys that other work-groups claimed, and hands every position its number.
// The last step waits for numbers that are not there yet.  Whoever claimed such a key is running, and
// writes its numbers before it waits for anybody else's, so every wait ends, provided that no other call works
// on the table.  One that does (a caller's mistake) can take a number away again: the wait is therefore bounded
// and ends with a flag (kMaxRounds).
// Bound by the chain of dependent round trips (key, swap, counter, number).  Two launches, the second
// looking every position up again, took 17.7 us of kernel time for 106,496 keys (44 % distinct); this took 12.1 us, 15.9
// with a load of the slot in front of each compare-and-swap, 38 with the line of the slot loaded beside it.  Per call, with the wipe on other
// work-groups and tables that are emptier: 11.9 -> 10.4 us, 32,000 keys of which none is there twice 17.7 -> 7.1.
// The order of unique_keys is the order in which tiles reach the counter: unspecified.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <new>
#include <string>

#include "hps_dedup.h"
#include "hps_dedup_missed.h"
#include "hps_mix.h"
#include "hps_rows.h"

namespace {

constexpr int64_t  kEmpty = INT64_MIN;            // free slot of both hash tables
constexpr int      kBlock = 256;
constexpr uint32_t kSmallBatch = 32768;           // most keys that go in tiles of 512 (launch_dedup)
constexpr uint64_t kMagic = 0x4850534445445550ull;
constexpr uint32_t kNone  = 0xFFFFFFFFu;
// Looks at a number that another work-group has to write, some 0.1 s of them; it is there after a few.
constexpr uint32_t kMaxRounds = 1u << 16;

// Scratch of hps_dedup_noalloc, the entry point for callers that cannot allocate: one hash table
// for batches of up to kNaMaxKeys keys (2 slots per key, 8-byte key word + 4-byte number per
// slot, one extra slot for the key that equals the free marker) and its counter words, in a
// static device array (3 MiB that every GPU the library runs on holds until the process ends).
constexpr uint32_t kNaMaxKeys  = HPS_DEDUP_NOALLOC_MAX;
constexpr uint32_t kNaSlots    = 2 * kNaMaxKeys;                        // a power of two
constexpr size_t   kNaKeyBytes = (((size_t)kNaSlots + 1) * 8 + 255) / 256 * 256;
constexpr size_t   kNaUidBytes = (((size_t)kNaSlots + 1) * 4 + 255) / 256 * 256;
constexpr size_t   kNaBytes    = kNaKeyBytes + kNaUidBytes + 256;       // + the counter, + the flag word
constexpr size_t   kFlagOffset = 64;                                    // of the flag word behind the (first) counter, in bytes
static_assert((kNaSlots & (kNaSlots - 1)) == 0, "slot count must be a power of two");
static __device__ __align__(256) unsigned char scratch[kNaBytes];

constexpr int kNaMaxDevices = 64;
std::mutex g_na_mu;
unsigned char *g_na_ptr[kNaMaxDevices];          // device address of `scratch` on each device, once known

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

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

__device__ __forceinline__ uint32_t bits_below(uint64_t m) {         // set bits of m below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The table has slots 0..mask for ordinary keys and slot mask + 1 for the key whose value is the
// free-slot marker itself.  Clears a whole table and the counter of its calls.
__global__ void dedup_clear_kernel(int64_t *tkey, uint32_t *tuid, uint64_t n_slots, uint64_t *counter) {
    const uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    for (uint64_t i = t; i < n_slots; i += (uint64_t)gridDim.x * blockDim.x) {
        tkey[i] = kEmpty;
        tuid[i] = kNone;
    }
    if (t == 0) *counter = 0ull;
}

__global__ void set_u32_kernel(uint32_t *p, uint32_t v) { *p = v; }

// A call's slots for n keys: a power of two, at least 2 * n; at least 4 * n up to 2^18 keys and 8 * n from 513 to 2^15, where wiping them is
// little and the unluckiest lane's attempts, one round trip each, are what the call waits for (us, at least 2 / 4 / 8 n: 2,000 distinct keys
// 11.0 / 7.0 / 5.9, 32,000 15.5 / 8.6 / 7.1, 106,496 17.7 / 12.8, of which 38,600 distinct 11.2 / 10.6; 65,000 4 / 8 n 10.8 / 10.9).  Up to 512
// keys stay in 1,024 slots, which a test fills to the last one.
__host__ __device__ __forceinline__ uint64_t slots_for(uint64_t n) {
    const uint64_t least = n <= 512 ? 2 * n : n <= (1u << 15) ? 8 * n : n <= (1u << 18) ? 4 * n : 2 * n;
    uint64_t p = 1024;
    while (p < least) p <<= 1;
    return p;
}

// Arguments that arrive in registers, in vectors (see hps_cache.hip), and the others.
typedef uint64_t u64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <typename T> __device__ __forceinline__ T *global_at(uint64_t word) { return (T *)(__attribute__((address_space(1))) T *)word; }
inline uint64_t word_of(const void *p) { return (uint64_t)reinterpret_cast<uintptr_t>(p); }
struct DedupArgs {
    uint32_t *flags;
    int64_t  *unique_keys;
    uint32_t *inverse, *n_unique;
    int64_t  *other_tkey;        // the table that the previous call worked on: its first other_dirty slots
    uint32_t *other_tuid;
    uint64_t  other_dirty;
    uint32_t  groups;            // work-groups of the launch
    // what hps_dedup_missed adds to a call
    const uint32_t *n_dev;       // the batch's length (<= n)
    uint32_t *n_host;            // it goes here too
    int64_t  *keys_host;         // and unique_keys here
};

// counter: low half = distinct keys so far, high half = tiles that have added theirs; zero between calls.
// Work-groups 0 .. tiles - 1 take a tile of keys each; those from `wipers` on wipe the other table, a tile's behind its keys.
template <int kTile, bool kMissed>                                   // keys (= threads) per work-group
__global__ void __launch_bounds__(kTile) dedup_kernel(const u64x4 pointers, const u32x4 sizes, const DedupArgs a) {
    const int64_t *__restrict__ const keys = global_at<const int64_t>(pointers.x);
    int64_t *const tkey = global_at<int64_t>(pointers.y);
    uint32_t *const tuid = global_at<uint32_t>(pointers.z);
    uint64_t *const counter = global_at<uint64_t>(pointers.w);
    uint32_t n = sizes.x, mask = sizes.y;
    const uint32_t tiles = sizes.z;                    // of the longest batch there may be
    const uint32_t wipers = sizes.w;                   // the first work-group that wipes: tiles, or 0
    constexpr int kLds = 2 * kTile;                    // LDS table slots (load <= 0.5)
    __shared__ unsigned long long l_key[kLds];
    __shared__ uint32_t l_uid[kLds + 1];               // number of the key in that slot; the last one: of the marker
    __shared__ uint32_t l_marker_seen, l_cnt, l_base;

    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t tile = blockIdx.x;
    auto wipe = [&] {
        for (uint64_t i = (uint64_t)(tile - wipers) * kTile + threadIdx.x; i < a.other_dirty; i += (uint64_t)(a.groups - wipers) * kTile) {
            a.other_tkey[i] = kEmpty;
            a.other_tuid[i] = kNone;
        }
    };
    if (tile >= tiles) return wipe();
    const uint32_t i = tile * kTile + threadIdx.x;
    const int64_t key = i < n ? keys[i] : 0;           // (of a length that is on the device: requested beside it)
    if (kMissed) {
        const uint32_t nd = *a.n_dev;
        n = nd < n ? nd : n;
        mask = (uint32_t)(slots_for(n) - 1);
        if (tile == 0 && threadIdx.x == 0) {
            *a.n_host = n;
            if (n == 0) *a.n_unique = 0u;              // no tile does
        }
        if ((uint64_t)tile * kTile >= n) {
            if (wipers == 0u) wipe();
            return;
        }
    }
    const uint32_t n_tiles = (n + kTile - 1) / kTile;
    const bool live = i < n;
    for (uint32_t j = threadIdx.x; j < (uint32_t)kLds; j += kTile) l_key[j] = (unsigned long long)kEmpty;
    if (threadIdx.x == 0) {
        l_marker_seen = 0u;
        l_cnt = 0u;
    }
    __syncthreads();

    // one lane per distinct key of the tile goes on
    const uint64_t h = mix64((uint64_t)key);
    bool elected = false;
    uint32_t ls = (uint32_t)kLds;
    if (live) {
        if (key == kEmpty) {
            elected = atomicCAS(&l_marker_seen, 0u, 1u) == 0u;
        } else {
            ls = (uint32_t)(h >> 40) & (kLds - 1);
            for (;;) {
                const unsigned long long old =
                    atomicCAS(&l_key[ls], (unsigned long long)kEmpty, (unsigned long long)key);
                if (old == (unsigned long long)kEmpty) { elected = true; break; }
                if (old == (unsigned long long)key) break;
                ls = (ls + 1) & (kLds - 1);                // at most half of the slots are ever taken
            }
        }
    }
    // the elected lane claims the key's slot of the global table, or finds that another tile has it
    bool won = false, listed = false;                  // listed: another tile has the key's slot, its number is there or on its way
    uint32_t slot = 0u;
    auto claim = [&](uint32_t at, int64_t with) {
        const unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long *>(tkey + at), (unsigned long long)kEmpty, (unsigned long long)with);
        slot = at;
        won = old == (unsigned long long)kEmpty;
        listed = old == (unsigned long long)key;
    };
    if (elected && key == kEmpty) {
        claim(mask + 1u, 0);
        listed = !won;
    } else if (elected) {
        const uint32_t home = (uint32_t)h & mask;
        for (uint32_t j = 0; j <= mask; ++j) {                    // the table is at most half full
            claim((home + j) & mask, key);
            if (won || listed) break;
        }
    }
    const uint64_t wonmask = __ballot(won);
    uint32_t first = 0u;
    if (lane == 0 && wonmask) first = atomicAdd(&l_cnt, (uint32_t)__popcll(wonmask));
    const uint32_t rank = (uint32_t)__shfl((int)first, 0, 64) + bits_below(wonmask);
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint64_t old = __hip_atomic_fetch_add(counter, (1ull << 32) | (uint64_t)l_cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        l_base = (uint32_t)old;
        if ((uint32_t)(old >> 32) + 1u == n_tiles) {
            *a.n_unique = (uint32_t)old + l_cnt;
            __hip_atomic_store(counter, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (won) {
        const uint32_t uid = l_base + rank;
        __hip_atomic_store(tuid + slot, uid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a.unique_keys[uid] = key;
        if (kMissed) a.keys_host[uid] = key;
        l_uid[ls] = uid;
    }
    // Every number of this work-group is on its way: only now wait for the others'.  (The barrier also keeps the
    // compiler from making the two conditions the two sides of one branch, the waiting side first.)
    __syncthreads();
    if (elected && !won) {
        uint32_t uid = kNone;
        for (uint32_t round = 0; listed && round < kMaxRounds; ++round) {
            uid = __hip_atomic_load(tuid + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (uid != kNone) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (uid == kNone) {                                       // no number came, or the table has no room: say so
            __hip_atomic_fetch_or(a.flags, (uint32_t)HPS_DEDUP_FLAG_STUCK, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            uid = 0u;                                             // a place that an expansion may read
        }
        l_uid[ls] = uid;
    }
    __syncthreads();
    if (live) a.inverse[i] = l_uid[ls];
    if (wipers == 0u) wipe();
}

}  // namespace

struct hps_dedup_session {
    uint64_t  magic;
    int       device;
    size_t    max_n;
    uint64_t  slots;        // slots_for(max_n); one more slot follows them
    int64_t  *tkey[3];      // [slots + 1] each; a call works on tkey[cur] (0 or 1), which is all free;
                            // table 2 serves calls that are being captured into a graph (see hps_dedup)
    uint32_t *tuid[3];      // [slots + 1] each
    uint64_t *counter;      // one word for each of the tables, zero between calls; kFlagOffset bytes on the flag word
    uint64_t  dirty[2];     // leading slots of each table that a call has written and nobody cleared yet
    int       cur;
    int       n_cus;
};

namespace {

hps_status_t check_session(hps_dedup_session *s) {
    if (!s || s->magic != kMagic) return fail(HPS_ERR_INVALID_ARG, "not a live dedup session");
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != s->device) return fail(HPS_ERR_INVALID_ARG, "session belongs to another device than the current one");
    return HPS_OK;
}

// Keys per work-group: 1024; 512 for batches that would leave most CUs without a work-group, whose lanes then share
// LDS slots with half as many others (kernel times: 2,000 keys 7.7 -> 6.7 us, 16,000 9.1 -> 7.3, 32,000 9.3 -> 8.1, 65,000 equal).
//
// Work-groups: one per tile.  What the previous call has used of the other table is wiped by further ones while the tiles leave an eighth of the CUs
// free for them (up to kBeside keys), off the tiles' chain of round trips: 106,496 keys, 38,600 distinct, 11.9 -> 11.2 us.  Beyond, the tiles wipe when
// they are done (425,984 keys, none twice, 38.5 us; further work-groups beside them 40.4; 240,000 to 262,000 keys, a tenth distinct, 20.9 / 23.7, 44 % distinct 23.2 / 25.2, none
// twice 21.6 / 21.1, but 44 % of 200,000 to 229,000 19.7 / 18.4), and more work-groups if those would have to wipe more than
// kWipeBehind slots per thread (300 keys behind a call of 2^20: 284 us by its one tile, 12 this way).
constexpr uint32_t kWipe = 8, kWipeBehind = 4, kBeside = 7u << 15;

template <bool kMissed = false>
void launch_dedup(const int64_t *keys, uint32_t n, int64_t *tkey, uint32_t *tuid, uint32_t mask, uint64_t *counter, hipStream_t st, DedupArgs a) {
    const uint32_t tile = n <= kSmallBatch ? 512u : 1024u;
    const uint32_t tiles = (n + tile - 1) / tile;
    const bool beside = n <= kBeside;
    const uint32_t per = (beside ? kWipe : kWipeBehind) * tile;
    const uint32_t wiping = (uint32_t)((a.other_dirty + per - 1) / per);            // (at most 2^31 + 1 slots)
    a.groups = beside ? tiles + wiping : tiles > wiping ? tiles : wiping;
    const dim3 grid(a.groups), block(tile);
    const u64x4 pointers = {word_of(keys), word_of(tkey), word_of(tuid), word_of(counter)};
    const u32x4 sizes = {n, mask, tiles, beside ? tiles : 0u};
    if (tile == 512u) hipLaunchKernelGGL((dedup_kernel<512, kMissed>), grid, block, 0, st, pointers, sizes, a);
    else              hipLaunchKernelGGL((dedup_kernel<1024, kMissed>), grid, block, 0, st, pointers, sizes, a);
}

uint32_t *flags_behind(uint64_t *counter) { return reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(counter) + kFlagOffset); }

// The array of hps_dedup_noalloc on device dev.  The array's name is only a host-side stand-in: its device address is
// asked for once per device (each GPU holds its own copy at its own address) and used from then on.
hps_status_t noalloc_base(int dev, unsigned char **base) {
    if (dev < 0 || dev >= kNaMaxDevices) return fail(HPS_ERR_INVALID_ARG, "device number beyond what hps_dedup_noalloc keeps track of");
    std::lock_guard<std::mutex> lk(g_na_mu);
    if (!g_na_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(HPS_ERR_DEVICE, "hipGetSymbolAddress returned no address for the scratch array");
        g_na_ptr[dev] = static_cast<unsigned char *>(p);
    }
    *base = g_na_ptr[dev];
    return HPS_OK;
}

}  // namespace

hps_status_t hps_dedup_missed(hps_dedup_session *s, const int64_t *keys, size_t n_max, const uint32_t *n_dev, int64_t *unique_keys,
                              int64_t *keys_host, uint32_t *inverse, uint32_t *n_host, uint32_t *n_unique, hipStream_t st) {
    if (hps_status_t e = check_session(s)) return e;
    if (n_max == 0 || n_max > s->max_n) return fail(HPS_ERR_INVALID_ARG, "n_max must be in 1 .. the session's max_n");
    const int t = s->cur, o = 1 - t;
    launch_dedup<true>(keys, (uint32_t)n_max, s->tkey[t], s->tuid[t], 0u, s->counter + t, st,
                       DedupArgs{flags_behind(s->counter), unique_keys, inverse, n_unique, s->tkey[o], s->tuid[o], s->dirty[o], 0u, n_dev, n_host, keys_host});
    HIP_TRY(hipGetLastError());
    s->dirty[t] = slots_for(n_max) + 1;
    s->dirty[o] = 0;
    s->cur = o;
    return HPS_OK;
}

void hps_dedup_missed_were(hps_dedup_session *s, size_t n) { s->dirty[1 - s->cur] = n ? slots_for(n) + 1 : 0; }

extern "C" {

const char *hps_dedup_last_error(void) { return g_err.c_str(); }

hps_status_t hps_dedup_create(size_t max_n, hps_dedup_t **out) {
    if (!out) return fail(HPS_ERR_INVALID_ARG, "out must not be NULL");
    *out = nullptr;
    // slots_for(max_n) must stay below 2^32: slot numbers, the mask and the extra slot behind the table are 32-bit
    if (max_n == 0 || max_n > (1ull << 30)) return fail(HPS_ERR_INVALID_ARG, "max_n must be in 1 .. 2^30");
    hps_dedup_session *s = new (std::nothrow) hps_dedup_session();
    if (!s) return fail(HPS_ERR_OOM, "host allocation failed");
    s->magic = 0;
    s->max_n = max_n;
    s->slots = slots_for(max_n);
    s->tkey[0] = s->tkey[1] = s->tkey[2] = nullptr;
    s->tuid[0] = s->tuid[1] = s->tuid[2] = nullptr;
    s->counter = nullptr;
    s->dirty[0] = s->dirty[1] = 0;
    s->cur = 0;
    s->n_cus = 256;
    hipError_t e = hipGetDevice(&s->device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&s->n_cus, hipDeviceAttributeMultiprocessorCount, s->device);
    if (e == hipSuccess && s->n_cus <= 0) s->n_cus = 256;
    for (int t = 0; t < 3; ++t) {
        if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void **>(&s->tkey[t]), (s->slots + 1) * sizeof(int64_t));
        if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void **>(&s->tuid[t]), (s->slots + 1) * sizeof(uint32_t));
    }
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void **>(&s->counter), 256);
    for (int t = 0; t < 3 && e == hipSuccess; ++t) {
        hipLaunchKernelGGL(dedup_clear_kernel, dim3(4096), dim3(kBlock), 0, 0, s->tkey[t], s->tuid[t], s->slots + 1,
                           s->counter + t);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(set_u32_kernel, dim3(1), dim3(1), 0, 0, flags_behind(s->counter), 0u);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(0);
    if (e != hipSuccess) {
        for (int t = 0; t < 3; ++t) {
            (void)hipFree(s->tkey[t]);
            (void)hipFree(s->tuid[t]);
        }
        (void)hipFree(s->counter);
        delete s;
        (void)hipGetLastError();
        return fail(e == hipErrorOutOfMemory ? HPS_ERR_OOM : HPS_ERR_DEVICE,
                    std::string("hps_dedup_create: ") + hipGetErrorString(e));
    }
    s->magic = kMagic;
    *out = s;
    return HPS_OK;
}

hps_status_t hps_dedup_destroy(hps_dedup_t *s) {
    if (!s) return HPS_OK;
    if (s->magic != kMagic) return fail(HPS_ERR_INVALID_ARG, "not a live dedup session");
    int prev = -1;
    HIP_TRY(hipGetDevice(&prev));
    HIP_TRY(hipSetDevice(s->device));
    hipError_t e = hipDeviceSynchronize();
    for (int t = 0; t < 3; ++t) {
        (void)hipFree(s->tkey[t]);
        (void)hipFree(s->tuid[t]);
    }
    (void)hipFree(s->counter);
    s->magic = 0;
    delete s;
    (void)hipSetDevice(prev);
    if (e != hipSuccess) return fail(HPS_ERR_DEVICE, std::string("hipDeviceSynchronize: ") + hipGetErrorString(e));
    return HPS_OK;
}

hps_status_t hps_dedup(hps_dedup_t *s, const int64_t *keys, size_t n, int64_t *unique_keys,
                       uint32_t *inverse, uint32_t *n_unique, void *stream) {
    if (hps_status_t st = check_session(s)) return st;
    if (!n_unique || !aligned(n_unique, 4)) return fail(HPS_ERR_INVALID_ARG, "n_unique must be a 4-byte aligned device pointer");
    if (n > s->max_n) return fail(HPS_ERR_INVALID_ARG, "n exceeds the session's max_n");
    hipStream_t q = static_cast<hipStream_t>(stream);
    if (n == 0) {
        hipLaunchKernelGGL(set_u32_kernel, dim3(1), dim3(1), 0, q, n_unique, 0u);
        HIP_TRY(hipGetLastError());
        return HPS_OK;
    }
    if (!keys || !unique_keys || !inverse) return fail(HPS_ERR_INVALID_ARG, "keys, unique_keys and inverse must not be NULL when n > 0");
    if (!aligned(keys, 8) || !aligned(unique_keys, 8) || !aligned(inverse, 4))
        return fail(HPS_ERR_INVALID_ARG, "keys and unique_keys must be 8-byte, inverse 4-byte aligned");
    const uint64_t slots = slots_for(n);            // <= s->slots because n <= max_n
    const uint32_t mask = (uint32_t)(slots - 1);
    const uint32_t cap = (uint32_t)s->n_cus * 8u;
    // A call that is being captured into a graph must be complete in itself, because the graph may
    // be replayed any number of times between other calls: it clears its own table (the third
    // one, which no other call touches) first and leaves the two alternating tables alone.
    hipStreamCaptureStatus cap_status = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing(q, &cap_status));
    if (cap_status != hipStreamCaptureStatusNone) {
        const uint64_t cb = (slots + 1 + kBlock - 1) / kBlock;
        hipLaunchKernelGGL(dedup_clear_kernel, dim3((uint32_t)(cb < cap ? cb : cap)), dim3(kBlock), 0, q,
                           s->tkey[2], s->tuid[2], slots + 1, s->counter + 2);
        launch_dedup(keys, (uint32_t)n, s->tkey[2], s->tuid[2], mask, s->counter + 2, q,
                     DedupArgs{flags_behind(s->counter), unique_keys, inverse, n_unique, nullptr, nullptr, 0, 0u, nullptr, nullptr, nullptr});
        HIP_TRY(hipGetLastError());
        return HPS_OK;
    }
    const int t = s->cur, o = 1 - t;
    launch_dedup(keys, (uint32_t)n, s->tkey[t], s->tuid[t], mask, s->counter + t, q,
                 DedupArgs{flags_behind(s->counter), unique_keys, inverse, n_unique, s->tkey[o], s->tuid[o], s->dirty[o], 0u, nullptr, nullptr, nullptr});
    HIP_TRY(hipGetLastError());
    s->dirty[t] = slots + 1;          // this call's slots, the extra one included
    s->dirty[o] = 0;
    s->cur = o;
    return HPS_OK;
}

hps_status_t hps_dedup_noalloc(const int64_t *keys, size_t n, int64_t *unique_keys, uint32_t *inverse,
                               uint32_t *n_unique, void *stream) {
    if (!n_unique || !aligned(n_unique, 4)) return fail(HPS_ERR_INVALID_ARG, "n_unique must be a 4-byte aligned device pointer");
    if (n > kNaMaxKeys)
        return fail(HPS_ERR_INVALID_ARG, "hps_dedup_noalloc takes at most " + std::to_string(kNaMaxKeys) +
                                             " keys per call (its table is a fixed static array); use a session of hps_dedup for more");
    hipStream_t q = static_cast<hipStream_t>(stream);
    if (n == 0) {
        hipLaunchKernelGGL(set_u32_kernel, dim3(1), dim3(1), 0, q, n_unique, 0u);
        HIP_TRY(hipGetLastError());
        return HPS_OK;
    }
    if (!keys || !unique_keys || !inverse) return fail(HPS_ERR_INVALID_ARG, "keys, unique_keys and inverse must not be NULL when n > 0");
    if (!aligned(keys, 8) || !aligned(unique_keys, 8) || !aligned(inverse, 4))
        return fail(HPS_ERR_INVALID_ARG, "keys and unique_keys must be 8-byte, inverse 4-byte aligned");
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    unsigned char *base = nullptr;
    if (hps_status_t st = noalloc_base(dev, &base)) return st;
    int64_t  *tkey    = reinterpret_cast<int64_t *>(base);
    uint32_t *tuid    = reinterpret_cast<uint32_t *>(base + kNaKeyBytes);
    uint64_t *counter = reinterpret_cast<uint64_t *>(base + kNaKeyBytes + kNaUidBytes);
    int n_cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (n_cus <= 0) n_cus = 256;
    const uint64_t slots = slots_for(n) < kNaSlots ? slots_for(n) : kNaSlots;      // >= 2 n because n <= kNaMaxKeys
    const uint32_t mask = (uint32_t)(slots - 1);
    const uint32_t cap = (uint32_t)n_cus * 8u;
    // The array keeps what the last call left in it: the slots this call may touch and its counter
    // are cleared first (by a kernel, so that the call can be captured into a graph).
    const uint64_t cb = (slots + 1 + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(dedup_clear_kernel, dim3((uint32_t)(cb < cap ? cb : cap)), dim3(kBlock), 0, q, tkey, tuid, slots + 1, counter);
    launch_dedup(keys, (uint32_t)n, tkey, tuid, mask, counter, q,
                 DedupArgs{flags_behind(counter), unique_keys, inverse, n_unique, nullptr, nullptr, 0, 0u, nullptr, nullptr, nullptr});
    HIP_TRY(hipGetLastError());
    return HPS_OK;
}

hps_status_t hps_dedup_flags(hps_dedup_t *s, uint32_t *flags, int clear) {
    if (!flags) return fail(HPS_ERR_INVALID_ARG, "flags is NULL");
    uint32_t *word = nullptr;
    if (s) {
        if (hps_status_t st = check_session(s)) return st;
        word = flags_behind(s->counter);
    } else {
        int dev = -1;
        HIP_TRY(hipGetDevice(&dev));
        unsigned char *base = nullptr;
        if (hps_status_t st = noalloc_base(dev, &base)) return st;
        word = flags_behind(reinterpret_cast<uint64_t *>(base + kNaKeyBytes + kNaUidBytes));
    }
    HIP_TRY(hipMemcpy(flags, word, sizeof(uint32_t), hipMemcpyDeviceToHost));
    const uint32_t zero = 0u;
    if (clear) HIP_TRY(hipMemcpy(word, &zero, sizeof(uint32_t), hipMemcpyHostToDevice));
    return HPS_OK;
}

hps_status_t hps_dedup_debug_claim(hps_dedup_t *s, int64_t key, size_t n) {
    if (hps_status_t st = check_session(s)) return st;
    if (n == 0 || n > s->max_n) return fail(HPS_ERR_INVALID_ARG, "n must be in 1 .. max_n");
    const uint64_t mask = slots_for(n) - 1;
    int64_t *tkey = s->tkey[s->cur];
    HIP_TRY(hipDeviceSynchronize());
    if (key == kEmpty) {                               // its slot holds anything but the marker
        const int64_t taken = 0;
        HIP_TRY(hipMemcpy(tkey + mask + 1, &taken, sizeof(taken), hipMemcpyHostToDevice));
        return HPS_OK;
    }
    for (uint64_t probe = 0, slot = mix64((uint64_t)key) & mask; probe <= mask; ++probe, slot = (slot + 1) & mask) {
        int64_t there = 0;
        HIP_TRY(hipMemcpy(&there, tkey + slot, sizeof(there), hipMemcpyDeviceToHost));
        if (there != kEmpty) continue;
        HIP_TRY(hipMemcpy(tkey + slot, &key, sizeof(key), hipMemcpyHostToDevice));
        return HPS_OK;
    }
    return fail(HPS_ERR_INVALID_ARG, "the table has no free slot");
}

hps_status_t hps_expand_rows(const float *rows, const uint32_t *inverse, size_t n, uint32_t dim,
                             float *out, void *stream) {
    if (dim == 0 || dim % 4 != 0) return fail(HPS_ERR_INVALID_ARG, "dim must be a non-zero multiple of 4");
    if (n == 0) return HPS_OK;
    if (n >= (1ull << 32)) return fail(HPS_ERR_INVALID_ARG, "n must be < 2^32");
    if (!rows || !inverse || !out) return fail(HPS_ERR_INVALID_ARG, "rows, inverse and out must not be NULL when n > 0");
    if (!aligned(rows, 16) || !aligned(out, 16) || !aligned(inverse, 4))
        return fail(HPS_ERR_INVALID_ARG, "rows and out must be 16-byte, inverse 4-byte aligned");
    int dev = -1, cus = 0;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    HIP_TRY(hps_launch_expand_rows(rows, inverse, (uint32_t)n, dim, out, cus > 0 ? (uint32_t)cus : 256u, static_cast<hipStream_t>(stream)));
    return HPS_OK;
}

}  // extern "C"

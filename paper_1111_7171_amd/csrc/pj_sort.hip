// pj_sort.hip -- device-wide primitives of libpassjoin: exclusive scan, stable radix sort,
// ordered compaction of run heads.
//
// Each is one pass over its data: a block takes a tile in order (a ticket), publishes the tile's
// total, and finds the totals of the tiles before it by looking back over what they published.
// A status word holds a total and whether it is the tile's own (kOwn) or includes every tile
// before it (kAll); it is stored and read with relaxed agent-scope atomics, and the word is all
// that passes between blocks, so no fence is needed.  A tile publishes its own total before it
// waits for any other, and a ticket is only taken by a running block, so every wait ends.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "pj_internal.h"
#include "pj_device_common.h"

namespace pj {

// ------------------------------------------------------------------------------------------
// Tile tickets and status words
// ------------------------------------------------------------------------------------------

// S is uint32_t where totals stay below 2^30, else uint64_t (totals below 2^62)
template <typename S>
struct Status {
    static constexpr int kShift = sizeof(S) * 8 - 2;
    static constexpr S kOwn = (S)1 << kShift, kAll = (S)2 << kShift;
    static constexpr S kMask = kOwn - 1;
    __device__ static inline S load(const S* p)
    {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ static inline void store(S* p, S v)
    {
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

__device__ inline uint32_t take_ticket(uint32_t* ticket, uint32_t* s_tile)
{
    if (threadIdx.x == 0) *s_tile = atomicAdd(ticket, 1u);
    __syncthreads();
    return *s_tile;
}

// Sum of the tiles before `tile`, found by the calling wave 64 predecessors at a time (a lane
// each); every lane returns it.
template <typename S>
__device__ inline S wave_look_back(const S* status, uint32_t tile)
{
    const int lane = threadIdx.x & 63;
    S sum = 0;
    int64_t top = (int64_t)tile - 1;               // nearest predecessor not yet added
    while (top >= 0) {
        const int64_t t = top - lane;
        S v = t >= 0 ? Status<S>::load(status + t) : Status<S>::kAll;
        const uint64_t all = __ballot((v & Status<S>::kAll) != 0);
        const uint64_t none = __ballot((v & ~Status<S>::kMask) == 0);
        const int stop = all ? __ffsll((unsigned long long)all) - 1 : 63;
        // every predecessor up to the first complete one has to be published
        if (none & (stop == 63 ? ~0ull : (2ull << stop) - 1ull)) {
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        sum += wave_sum<S>(lane <= stop ? (S)(v & Status<S>::kMask) : (S)0);
        if (all) break;
        top -= 64;
    }
    return sum;
}

// ------------------------------------------------------------------------------------------
// Exclusive scan
// ------------------------------------------------------------------------------------------

constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;

// tmp: [ticket (16 bytes) | one 64-bit status word per tile], zeroed by the caller; one tile
// needs neither (look == nullptr)
template <typename TI, typename TO>
__global__ __launch_bounds__(kBlock) void k_scan(const TI* __restrict__ in, TO* __restrict__ out,
                                                 uint64_t n, uint32_t* ticket, uint64_t* look)
{
    __shared__ TO s_wave[kWaves];
    __shared__ uint64_t s_before;
    __shared__ uint32_t s_tile;
    const uint32_t tile = look ? take_ticket(ticket, &s_tile) : 0u;
    const uint64_t base = (uint64_t)tile * kScanTile + (uint64_t)threadIdx.x * kScanItems;
    TO v[kScanItems];
    TO sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? (TO)in[base + k] : 0;
        sum += v[k];
    }
    TO tot;
    TO run = block_excl_scan<TO>(sum, s_wave, &tot);
    if (look) {
        if (threadIdx.x < 64) {
            using W = Status<uint64_t>;
            if (threadIdx.x == 0) W::store(look + tile, (tile ? W::kOwn : W::kAll) | (uint64_t)tot);
            const uint64_t before = wave_look_back<uint64_t>(look, tile);
            if (threadIdx.x == 0) {
                s_before = before;
                if (tile) W::store(look + tile, W::kAll | ((before + (uint64_t)tot) & W::kMask));
            }
        }
        __syncthreads();
        run += (TO)s_before;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
    // the thread holding the last element writes the total
    if (n > 0 && base <= n - 1 && n - 1 < base + kScanItems) out[n] = run;
}

size_t scan_tmp_bytes(uint64_t n)
{
    const uint64_t nb = (n + kScanTile - 1) / kScanTile;
    return 16 + (size_t)nb * sizeof(uint64_t);
}

template <typename TO>
__global__ void k_zero_one(TO* __restrict__ out)
{
    if (threadIdx.x == 0) *out = 0;
}

template <typename TI, typename TO>
static hipError_t scan_impl(const TI* in, TO* out, uint64_t n, void* tmp, size_t tmp_bytes,
                            hipStream_t s)
{
    if (n == 0) {
        // a kernel, not a memset, so that the call can be captured in a graph
        hipLaunchKernelGGL((k_zero_one<TO>), dim3(1), dim3(64), 0, s, out);
        return hipGetLastError();
    }
    const uint64_t nb = (n + kScanTile - 1) / kScanTile;
    if (tmp_bytes < scan_tmp_bytes(n)) return hipErrorInvalidValue;
    uint32_t* ticket = (uint32_t*)tmp;
    uint64_t* look = nb > 1 ? (uint64_t*)tmp + 2 : nullptr;
    if (look) {
        const hipError_t e = launch_fill_words(ticket, 4 + 2 * nb, 0u, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_scan<TI, TO>), dim3((unsigned)nb), dim3(kBlock), 0, s, in, out, n, ticket,
                       look);
    return hipGetLastError();
}

hipError_t scan_u32_to_u32(const uint32_t* in, uint32_t* out, uint64_t n, void* tmp,
                           size_t tmp_bytes, hipStream_t s)
{
    return scan_impl<uint32_t, uint32_t>(in, out, n, tmp, tmp_bytes, s);
}

hipError_t scan_u32_to_u64(const uint32_t* in, unsigned long long* out, uint64_t n, void* tmp,
                           size_t tmp_bytes, hipStream_t s)
{
    return scan_impl<uint32_t, unsigned long long>(in, out, n, tmp, tmp_bytes, s);
}

// ------------------------------------------------------------------------------------------
// Stable LSD radix sort, 8-bit digits.  One kernel counts the digits of every pass (a key is
// read once for all of them); then a kernel a pass reads a tile, ranks its keys (a wave ranks
// its own 64 x ITEMS keys with ballots and wave-private counters, so there is no barrier per
// key), orders them in LDS by digit, finds where the tile's share of each digit begins by
// looking back, and writes every digit's keys as one run.  What bounds a pass is HBM for large
// inputs and the chain ticket -> rank -> look-back for small ones, so small inputs take small
// tiles (more blocks, shorter chains).
// ------------------------------------------------------------------------------------------

constexpr int kRadixPasses = 8;                   // digits of a 64-bit key
// Tile shapes (threads x keys a thread).  Measured for 46 bits with values (6 passes): 2x10^6
// entries 174 us with 512 x 8, 182 with 256 x 16, 233 with 256 x 8; 262,144 entries 83-86 us with
// every shape; 30,000 entries 58 us with 256 x 4, 62 with 256 x 8.  Keys alone leave LDS for tiles
// of 512 x 16: 65x10^6 keys of 40 bits 1.64 ms, against 2.15 with 512 x 8.  (A kernel each for
// counting, scanning and scattering a pass took 270 us and 2.9 ms for the first and the last.)
constexpr uint64_t kSmallSort = 1ull << 18, kLargeSort = 1ull << 23;
constexpr int kSmallT = 256, kSmallItems = 4;
constexpr int kMidT = 512, kMidItems = 8;
constexpr int kLargeT = 512, kLargeItems = 16;
constexpr int kLook = 8;                          // predecessors read at a time (4, 16: the same)

int radix_passes(int bits) { return bits <= 0 ? 0 : (bits + 7) / 8; }

static uint64_t radix_tile(uint64_t n, bool vals)
{
    return n < kSmallSort ? kSmallT * kSmallItems
                          : vals || n < kLargeSort ? kMidT * kMidItems : kLargeT * kLargeItems;
}

// head of the scratch: the digit counts of every pass and a ticket a pass, zeroed before the
// counting kernel; then two sets of status words (256 a tile), used by the passes in turn: a
// pass clears the set that the next one uses, the counting kernel the first one
constexpr uint64_t kRadixHead = kRadixPasses * 256 + 16;

template <typename K>
__global__ __launch_bounds__(kBlock) void k_radix_count(const K* __restrict__ keys, uint64_t n,
                                                        int passes, uint32_t* __restrict__ hist,
                                                        uint32_t* __restrict__ clear,
                                                        uint64_t clear_words)
{
    __shared__ uint32_t cnt[kRadixPasses][256];
    for (int p = 0; p < passes; ++p) cnt[p][threadIdx.x] = 0;
    __syncthreads();
    const uint64_t step = (uint64_t)gridDim.x * kBlock;
    const uint64_t t0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    for (uint64_t k = t0; k < clear_words; k += step) clear[k] = 0;
    for (uint64_t k0 = t0; k0 < n; k0 += 4 * step) {
        K key[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) key[u] = k0 + u * step < n ? keys[k0 + u * step] : (K)0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (k0 + u * step >= n) break;
            for (int p = 0; p < passes; ++p) {
                const uint32_t d = (uint32_t)(key[u] >> (8 * p)) & 255u;
                // keys in an order of their own often share a digit throughout the wave
                const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
                if (__ballot(d != d0) == 0) {
                    const uint64_t act = __ballot(true);
                    if ((act & lanemask_lt()) == 0) atomicAdd(&cnt[p][d0], (uint32_t)__popcll(act));
                } else {
                    atomicAdd(&cnt[p][d], 1u);
                }
            }
        }
    }
    __syncthreads();
    for (int p = 0; p < passes; ++p)
        if (cnt[p][threadIdx.x]) atomicAdd(&hist[p * 256 + threadIdx.x], cnt[p][threadIdx.x]);
}

// Where a pass takes entry k from: arrays, or (LengthSource) string k's length and its id.
template <typename K>
struct ArraySource {
    const K* keys;
    const uint32_t* vals;
    __device__ inline K key(uint64_t k) const { return keys[k]; }
    __device__ inline uint32_t val(uint64_t k) const { return vals[k]; }
};
struct LengthSource {
    const int32_t* offs;
    __device__ inline uint32_t key(uint64_t k) const { return (uint32_t)(offs[k + 1] - offs[k]); }
    __device__ inline uint32_t val(uint64_t k) const { return (uint32_t)k; }
};

// keys_out may be nullptr (the keys are not wanted)
template <typename K, typename S, int T, int ITEMS, bool VALS, typename Source>
__global__ __launch_bounds__(T) void k_radix_pass(Source src, uint64_t n,
                                                  int shift, const uint32_t* __restrict__ hist,
                                                  uint32_t* ticket, S* look,
                                                  S* __restrict__ look_next,
                                                  K* __restrict__ keys_out,
                                                  uint32_t* __restrict__ vals_out)
{
    static_assert(T >= 256 && T % 64 == 0, "a thread per digit");
    constexpr int TILE = T * ITEMS, NW = T / 64;
    __shared__ K s_keys[TILE];
    __shared__ uint32_t s_vals[VALS ? TILE : 1];
    __shared__ uint32_t s_cnt[NW][256];
    __shared__ uint32_t s_dst[256];
    __shared__ uint32_t s_part[2][4];
    __shared__ uint32_t s_tile;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int k = threadIdx.x; k < NW * 256; k += T) (&s_cnt[0][0])[k] = 0;
    const uint32_t tile = take_ticket(ticket, &s_tile);
    const uint64_t base = (uint64_t)tile * TILE;
    const uint64_t wbase = base + (uint64_t)w * (64 * ITEMS) + (uint64_t)lane;
    K key[ITEMS];
    uint32_t val[VALS ? ITEMS : 1], rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint64_t idx = wbase + 64 * r;
        key[r] = idx < n ? src.key(idx) : (K)0;
        if (VALS) val[r] = idx < n ? src.val(idx) : 0u;
    }
    if (look_next && threadIdx.x < 256) look_next[(uint64_t)tile * 256 + threadIdx.x] = 0;
    // ranks within the wave's keys of one digit, in input order
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = wbase + 64 * r < n;
        const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint64_t bb = __ballot((d >> bit) & 1u);
            peers &= ((d >> bit) & 1u) ? bb : ~bb;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lanemask_lt());
        const uint32_t seen = s_cnt[w][d];
        rank[r] = seen + before;
        // the counter is read by every peer before the first of them moves it on (a wave's LDS
        // requests complete in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) s_cnt[w][d] = seen + (uint32_t)__popcll(peers);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread d < 256: the tile's keys of digit d, where each wave's begin, and where the digit
    // begins in the tile and in the output
    const bool digit = threadIdx.x < 256;
    uint32_t cw[NW], total = 0, lsum = 0, gsum = 0, gcnt = 0;
    S* mine = look + (uint64_t)tile * 256 + threadIdx.x;
    if (digit) {
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            cw[k] = total;
            total += s_cnt[k][threadIdx.x];
        }
        Status<S>::store(mine, (tile ? Status<S>::kOwn : Status<S>::kAll) | (S)total);
        gcnt = hist[threadIdx.x];
        lsum = wave_incl_scan(total);
        gsum = wave_incl_scan(gcnt);
        if (lane == 63) {
            s_part[0][w] = lsum;
            s_part[1][w] = gsum;
        }
    }
    __syncthreads();
    uint32_t local = lsum - total, begin = gsum - gcnt;
    if (digit) {
        for (int k = 0; k < w; ++k) {
            local += s_part[0][k];
            begin += s_part[1][k];
        }
#pragma unroll
        for (int k = 0; k < NW; ++k) s_cnt[k][threadIdx.x] = local + cw[k];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (wbase + 64 * r < n) {
            const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
            const uint32_t at = s_cnt[w][d] + rank[r];
            s_keys[at] = key[r];
            if (VALS) s_vals[at] = val[r];
        }
    }
    // the digit's keys in the tiles before, kLook predecessors read at a time
    if (digit) {
        S before = 0;
        for (int64_t t = (int64_t)tile - 1; t >= 0;) {
            S v[kLook];
#pragma unroll
            for (int k = 0; k < kLook; ++k)
                v[k] = t - k >= 0 ? Status<S>::load(look + (uint64_t)(t - k) * 256 + threadIdx.x)
                                  : Status<S>::kAll;
            bool done = false, wait = false;
#pragma unroll
            for (int k = 0; k < kLook; ++k) {
                wait = wait || (v[k] & ~Status<S>::kMask) == 0;
                if (!done && !wait) {
                    before += v[k] & Status<S>::kMask;
                    done = (v[k] & Status<S>::kAll) != 0;
                    --t;
                }
            }
            if (done) break;
            if (wait) __builtin_amdgcn_s_sleep(1);
        }
        if (tile) Status<S>::store(mine, Status<S>::kAll | ((before + (S)total) & Status<S>::kMask));
        s_dst[threadIdx.x] = begin + (uint32_t)before - local;     // n < 2^32: exact modulo 2^32
    }
    __syncthreads();
    const uint32_t m = (uint32_t)(n - base < (uint64_t)TILE ? n - base : (uint64_t)TILE);
    for (uint32_t j = threadIdx.x; j < m; j += T) {
        const K k = s_keys[j];
        const uint32_t o = s_dst[(uint32_t)(k >> shift) & 255u] + j;
        if (keys_out) keys_out[o] = k;
        if (VALS) vals_out[o] = s_vals[j];
    }
}

size_t radix_tmp_bytes(uint64_t n)
{
    const uint64_t tile = radix_tile(n, true);     // no larger than without values
    const uint64_t nt = (n + tile - 1) / tile;
    const size_t word = n < (1ull << 30) ? sizeof(uint32_t) : sizeof(uint64_t);
    return (size_t)kRadixHead * sizeof(uint32_t) + (size_t)(2 * nt * 256) * word + 256;
}

template <typename K, typename S>
static hipError_t radix_impl(K* keys, uint32_t* vals, K* keys_alt, uint32_t* vals_alt,
                             uint64_t n, int bits, void* tmp, bool* in_alt, hipStream_t s)
{
    const uint64_t tile = radix_tile(n, vals != nullptr);
    const uint64_t nt = (n + tile - 1) / tile;
    const int passes = radix_passes(bits);
    uint32_t* hist = (uint32_t*)tmp;
    uint32_t* tickets = hist + kRadixPasses * 256;
    S* look[2] = {(S*)(hist + kRadixHead), (S*)(hist + kRadixHead) + nt * 256};
    hipError_t e = launch_fill_words(hist, kRadixHead, 0u, s);
    if (e != hipSuccess) return e;
    // a block adds up to 256 counts a pass to the shared ones, so it takes thousands of keys
    const uint64_t per = n < kSmallSort ? 1024 : 4096;
    const unsigned cgrid = (unsigned)std::min<uint64_t>((n + per - 1) / per, 1024);
    hipLaunchKernelGGL((k_radix_count<K>), dim3(cgrid), dim3(kBlock), 0, s, keys, n, passes, hist,
                       (uint32_t*)look[0], nt * 256 * (sizeof(S) / 4));
    K* kin = keys; uint32_t* vin = vals;
    K* kout = keys_alt; uint32_t* vout = vals_alt;
    for (int p = 0; p < passes; ++p) {
        const ArraySource<K> src{kin, vin};
#define PJ_RADIX(T, ITEMS)                                                                        \
    do {                                                                                          \
        if (vals)                                                                                 \
            hipLaunchKernelGGL((k_radix_pass<K, S, T, ITEMS, true, ArraySource<K>>),              \
                               dim3((unsigned)nt), dim3(T), 0, s, src, n, 8 * p, hist + 256 * p,  \
                               tickets + p,                                                       \
                               look[p & 1], look[(p + 1) & 1], kout, vout);                       \
        else                                                                                      \
            hipLaunchKernelGGL((k_radix_pass<K, S, T, ITEMS, false, ArraySource<K>>),             \
                               dim3((unsigned)nt), dim3(T), 0, s, src, n, 8 * p, hist + 256 * p,  \
                               tickets + p,                                                       \
                               look[p & 1], look[(p + 1) & 1], kout, vout);                       \
    } while (0)
        if (n < kSmallSort) PJ_RADIX(kSmallT, kSmallItems);
        else if (vals || n < kLargeSort) PJ_RADIX(kMidT, kMidItems);
        else hipLaunchKernelGGL((k_radix_pass<K, S, kLargeT, kLargeItems, false, ArraySource<K>>),
                                dim3((unsigned)nt), dim3(kLargeT), 0, s, src, n, 8 * p,
                                hist + 256 * p, tickets + p, look[p & 1], look[(p + 1) & 1], kout,
                                vout);
#undef PJ_RADIX
        std::swap(kin, kout);
        std::swap(vin, vout);
        *in_alt = !*in_alt;
    }
    return hipGetLastError();
}

template <typename K>
static hipError_t radix_sort(K* keys, uint32_t* vals, K* keys_alt, uint32_t* vals_alt, uint64_t n,
                             int bits, void* tmp, size_t tmp_bytes, bool* in_alt, hipStream_t s)
{
    *in_alt = false;
    if (bits <= 0 || n == 0) return hipSuccess;
    if (bits > (int)sizeof(K) * 8 || n >= (1ull << 32) || tmp_bytes < radix_tmp_bytes(n))
        return hipErrorInvalidValue;
    if (n < (1ull << 30))
        return radix_impl<K, uint32_t>(keys, vals, keys_alt, vals_alt, n, bits, tmp, in_alt, s);
    return radix_impl<K, uint64_t>(keys, vals, keys_alt, vals_alt, n, bits, tmp, in_alt, s);
}

// Lengths below 256 are one digit, read from the offsets, and its counts are the length histogram
// that the set has already: one pass, without the key arrays and the counting kernel (10^6 strings:
// 18 us in place of 38).  The status words and the ticket are cleared first.
hipError_t launch_length_sort(const int32_t* offs, int64_t n, const int32_t* hist, int32_t* perm,
                              void* tmp, size_t tmp_bytes, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const uint64_t m = (uint64_t)n, tile = radix_tile(m, true), nt = (m + tile - 1) / tile;
    if (tmp_bytes < radix_tmp_bytes(m) || m >= (1ull << 31)) return hipErrorInvalidValue;
    // [ticket (16 bytes) | 256 status words a tile]; totals below 2^30 take 32-bit words
    const bool wide = m >= (1ull << 30);
    uint32_t* ticket = (uint32_t*)tmp;
    void* look = ticket + 4;
    hipError_t e = launch_fill_words(ticket, 4 + nt * 256 * (wide ? 2 : 1), 0u, s);
    if (e != hipSuccess) return e;
    const LengthSource src{offs};
#define PJ_LENGTHS(S, T, ITEMS)                                                                    \
    hipLaunchKernelGGL((k_radix_pass<uint32_t, S, T, ITEMS, true, LengthSource>),                  \
                       dim3((unsigned)nt), dim3(T), 0, s, src, m, 0, (const uint32_t*)hist, ticket, \
                       (S*)look, (S*)nullptr, (uint32_t*)nullptr, (uint32_t*)perm)
    if (m < kSmallSort) PJ_LENGTHS(uint32_t, kSmallT, kSmallItems);
    else if (!wide) PJ_LENGTHS(uint32_t, kMidT, kMidItems);
    else PJ_LENGTHS(uint64_t, kMidT, kMidItems);
#undef PJ_LENGTHS
    return hipGetLastError();
}

hipError_t radix_sort_u64(uint64_t* keys, uint32_t* vals, uint64_t* keys_alt, uint32_t* vals_alt,
                          uint64_t n, int bits, void* tmp, size_t tmp_bytes, bool* in_alt,
                          hipStream_t s)
{
    return radix_sort<uint64_t>(keys, vals, keys_alt, vals_alt, n, bits, tmp, tmp_bytes, in_alt, s);
}

hipError_t radix_sort_u32(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                          uint64_t n, int bits, void* tmp, size_t tmp_bytes, bool* in_alt,
                          hipStream_t s)
{
    return radix_sort<uint32_t>(keys, vals, keys_alt, vals_alt, n, bits, tmp, tmp_bytes, in_alt, s);
}

// ------------------------------------------------------------------------------------------
// Ordered compaction of the heads of runs of equal keys (one pass over the sorted keys)
// ------------------------------------------------------------------------------------------

constexpr int kHeadT = 512, kHeadItems = 16, kHeadTile = kHeadT * kHeadItems;

// f(position among the heads, index, key) for every head, in order; *count = their number.
// Element r * kHeadT + tid of a tile belongs to thread tid, so the reads are coalesced.
template <typename F>
__global__ __launch_bounds__(kHeadT) void k_compact_heads(const uint64_t* __restrict__ keys,
                                                          uint64_t n, uint32_t* ticket,
                                                          uint64_t* look,
                                                          uint32_t* __restrict__ count, F f)
{
    constexpr int kParts = kHeadItems * (kHeadT / 64);     // waves x rounds, in element order
    static_assert(kParts <= 128, "two parts a lane");
    __shared__ uint32_t s_part[kParts];
    __shared__ uint64_t s_before;
    __shared__ uint32_t s_tile;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t tile = look ? take_ticket(ticket, &s_tile) : 0u;
    const uint64_t base = (uint64_t)tile * kHeadTile + threadIdx.x;
    uint64_t key[kHeadItems];
    uint32_t heads = 0, rank[kHeadItems];
#pragma unroll
    for (int r = 0; r < kHeadItems; ++r) {
        const uint64_t k = base + (uint64_t)r * kHeadT;
        bool head = false;
        key[r] = 0;
        if (k < n) {
            key[r] = keys[k];
            head = k == 0 || keys[k - 1] != key[r];
        }
        const uint64_t m = __ballot(head);
        rank[r] = (uint32_t)__popcll(m & lanemask_lt());
        heads |= head ? 1u << r : 0u;
        if (lane == 0) s_part[r * (kHeadT / 64) + w] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    // wave 0: exclusive scan of the parts, then the tiles before
    if (threadIdx.x < 64) {
        const uint32_t p0 = 2 * lane < kParts ? s_part[2 * lane] : 0u;
        const uint32_t p1 = 2 * lane + 1 < kParts ? s_part[2 * lane + 1] : 0u;
        const uint32_t incl = wave_incl_scan(p0 + p1);
        const uint32_t total = __shfl(incl, 63, 64);
        if (2 * lane < kParts) s_part[2 * lane] = incl - p0 - p1;
        if (2 * lane + 1 < kParts) s_part[2 * lane + 1] = incl - p1;
        using W = Status<uint64_t>;
        uint64_t before = 0;
        if (look) {
            if (lane == 0) W::store(look + tile, (tile ? W::kOwn : W::kAll) | (uint64_t)total);
            before = wave_look_back<uint64_t>(look, tile);
            if (lane == 0 && tile) W::store(look + tile, W::kAll | (before + total));
        }
        if (lane == 0) {
            s_before = before;
            if ((uint64_t)tile * kHeadTile + kHeadTile >= n) *count = (uint32_t)(before + total);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kHeadItems; ++r)
        if ((heads >> r) & 1u)
            f((uint32_t)s_before + s_part[r * (kHeadT / 64) + w] + rank[r], base + (uint64_t)r * kHeadT,
              key[r]);
}

template <typename F>
static hipError_t compact_heads(const uint64_t* keys, uint64_t n, void* tmp, size_t tmp_bytes,
                                uint32_t* count, F f, hipStream_t s)
{
    if (n == 0) {
        hipLaunchKernelGGL((k_zero_one<uint32_t>), dim3(1), dim3(64), 0, s, count);
        return hipGetLastError();
    }
    const uint64_t nb = (n + kHeadTile - 1) / kHeadTile;
    if (tmp_bytes < scan_tmp_bytes(n)) return hipErrorInvalidValue;
    uint32_t* ticket = (uint32_t*)tmp;
    uint64_t* look = nb > 1 ? (uint64_t*)tmp + 2 : nullptr;
    if (look) {
        const hipError_t e = launch_fill_words(ticket, 4 + 2 * nb, 0u, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_compact_heads<F>), dim3((unsigned)nb), dim3(kHeadT), 0, s, keys, n, ticket,
                       look, count, f);
    return hipGetLastError();
}

// first entry of every run
struct RunStartOp {
    uint32_t* runstart;
    __device__ inline void operator()(uint32_t at, uint64_t k, uint64_t) const
    {
        runstart[at] = (uint32_t)k;
    }
};

hipError_t launch_run_starts(const uint64_t* keys, uint64_t n, void* tmp, size_t tmp_bytes,
                             uint32_t* runstart, uint32_t* count, hipStream_t s)
{
    return compact_heads(keys, n, tmp, tmp_bytes, count, RunStartOp{runstart}, s);
}

// distinct sorted pair keys as id columns
struct PairOp {
    int32_t *a, *b;
    int bbits;
    __device__ inline void operator()(uint32_t at, uint64_t, uint64_t key) const
    {
        a[at] = (int32_t)(key >> bbits);
        b[at] = (int32_t)(key & ((1ull << bbits) - 1));
    }
};

hipError_t launch_unique_pairs(const uint64_t* keys, uint64_t n, int bbits, void* tmp,
                               size_t tmp_bytes, int32_t* a, int32_t* b, uint32_t* count,
                               hipStream_t s)
{
    return compact_heads(keys, n, tmp, tmp_bytes, count, PairOp{a, b, bbits}, s);
}

// Few accepted candidates (a query batch, a small join): one block maps them to pair keys, sorts
// them in LDS (bitonic), drops repeats and writes the columns.  A step of the network costs a
// barrier, so past kSmallPairs keys the radix sort's launches cost less.
__global__ __launch_bounds__(1024) void k_small_pairs(const uint64_t* __restrict__ acc, uint32_t m,
                                                      const int32_t* __restrict__ xperm,
                                                      const int32_t* __restrict__ yperm, int self,
                                                      int bbits, int32_t* __restrict__ a,
                                                      int32_t* __restrict__ b,
                                                      uint32_t* __restrict__ count)
{
    __shared__ uint64_t s_k[kSmallPairs];
    __shared__ uint32_t s_w[16];
    uint32_t N = 64;
    while (N < m) N <<= 1;
    for (uint32_t k = threadIdx.x; k < N; k += 1024) {
        uint64_t key = ~0ull;
        if (k < m) {
            const uint64_t v = acc[k];
            uint32_t x = (uint32_t)xperm[v >> 32], y = (uint32_t)yperm[v & 0xffffffffu];
            if (self && y < x) { const uint32_t t = x; x = y; y = t; }
            key = ((uint64_t)x << bbits) | y;
        }
        s_k[k] = key;
    }
    __syncthreads();
    block_bitonic_sort(s_k, N, 1024u);
    uint32_t carry = 0;
    for (uint32_t base = 0; base < m; base += 1024) {
        const uint32_t k = base + threadIdx.x;
        const bool head = k < m && (k == 0 || s_k[k] != s_k[k - 1]);
        uint32_t tot;
        const uint32_t at = carry + block_rank_1024(head, s_w, &tot);
        if (head) {
            a[at] = (int32_t)(s_k[k] >> bbits);
            b[at] = (int32_t)(s_k[k] & ((1ull << bbits) - 1));
        }
        carry += tot;
    }
    if (threadIdx.x == 0) *count = carry;
}

hipError_t launch_small_pairs(const uint64_t* acc, uint64_t m, const int32_t* xperm,
                              const int32_t* yperm, int self, int bbits, int32_t* a, int32_t* b,
                              uint32_t* count, hipStream_t s)
{
    if (m > (uint64_t)kSmallPairs || bbits < 1 || bbits > 31) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_small_pairs, dim3(1), dim3(1024), 0, s, acc, (uint32_t)m, xperm, yperm, self,
                       bbits, a, b, count);
    return hipGetLastError();
}

}  // namespace pj

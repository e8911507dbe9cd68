// pj_device.hip -- gfx950 kernels of libpassjoin: arena, index, probe, verification, output.
//
// Everything here is integer work on wave64: no MFMA (nothing is a dense contraction).  The
// phases are HBM/L2-bound streaming (arena packing, index build, radix sort), random-access
// lookups (probe) and integer-VALU dynamic programming (verification).
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "pj_internal.h"
#include "pj_device_common.h"

namespace pj {

// ------------------------------------------------------------------------------------------
// String arena: length histogram + validation, (length, id) keys, packing
// ------------------------------------------------------------------------------------------

// Few blocks: each adds its counts to the shared ones, an atomic per length present (10^6 short
// strings: 46 us with a block per 256 strings, 9 us so)
__global__ __launch_bounds__(kBlock) void k_length_hist(const int32_t* __restrict__ offs,
                                                        int64_t n, int32_t* __restrict__ lcount)
{
    __shared__ int32_t h[kLenTab];
    for (int k = threadIdx.x; k < kLenTab; k += kBlock) h[k] = 0;
    __syncthreads();
    int32_t e = 0;
    for (int64_t id = (int64_t)blockIdx.x * kBlock + threadIdx.x; id < n;
         id += (int64_t)gridDim.x * kBlock) {
        const int32_t a = offs[id], b = offs[id + 1];
        if (id == 0 && a != 0) e |= 1;
        // the length as a 64-bit difference: offsets of any value are judged, not wrapped
        const int64_t l = (int64_t)b - (int64_t)a;
        if (l < 0) e |= 2;
        else if (l > kLenMax) e |= 4;
        else atomicAdd(&h[l], 1);
    }
    if (e) atomicOr(&lcount[kLenTab], e);
    __syncthreads();
    for (int k = threadIdx.x; k < kLenTab; k += kBlock)
        if (h[k]) atomicAdd(&lcount[k], h[k]);
}

// One block: the tables by length from the counts, strings and arena bytes before each length.
// (Uploads of host-made tables took the host 10-20 us each, with the device waiting; made by the last
// block of k_length_hist they cost that kernel 19 us for its fences.)  It also clears what the packing
// and the index fill in: the bitmap of bytes present and the codes.
__global__ __launch_bounds__(kBlock) void k_length_tables(const int32_t* __restrict__ lcount,
                                                          int32_t* __restrict__ lenstart,
                                                          int64_t* __restrict__ gbase,
                                                          uint32_t* __restrict__ bitmap,
                                                          uint16_t* __restrict__ code)
{
    __shared__ uint64_t s_wave[kWaves];
    if (bitmap) {
        if (threadIdx.x < 8) bitmap[threadIdx.x] = 0;
        code[threadIdx.x] = 0;
    }
    constexpr int kEach = (kLenTab + kBlock - 1) / kBlock;
    const int l0 = threadIdx.x * kEach;
    uint64_t strings = 0, bytes = 0, total;
    int32_t c[kEach];
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        c[k] = l0 + k < kLenTab ? lcount[l0 + k] : 0;
        strings += (uint64_t)c[k];
        bytes += (uint64_t)c[k] * (uint64_t)stride_of(l0 + k);
    }
    strings = block_excl_scan(strings, s_wave, &total);
    bytes = block_excl_scan(bytes, s_wave, &total);
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        if (l0 + k > kLenTab) break;
        lenstart[l0 + k] = (int32_t)strings;
        if (l0 + k < kLenTab) gbase[l0 + k] = (int64_t)bytes;
        strings += (uint64_t)c[k];
        bytes += (uint64_t)c[k] * (uint64_t)stride_of(l0 + k);
    }
}

__global__ __launch_bounds__(kBlock) void k_len_keys(const int32_t* __restrict__ offs, int64_t n,
                                                     uint32_t* __restrict__ keys,
                                                     uint32_t* __restrict__ vals)
{
    int64_t id = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (id < n) {
        keys[id] = (uint32_t)(offs[id + 1] - offs[id]);
        vals[id] = (uint32_t)id;
    }
}

// The strings in their padded slots of the sorted arena, 2^lps_shift lanes per string and 16 bytes
// a lane at a time (unaligned reads, aligned writes), and the byte values present: flags in LDS by
// block, added to the set's bitmap at the end.  A chunk that would read past the set's last byte is
// read byte by byte.  10^6 short strings: 59 us byte by byte and 37 for the byte values in a pass
// of their own, 32 us so (48 with a tested bit for each byte in place of the flags).
struct __attribute__((packed)) Unaligned16 {
    uint32_t w[4];
};

__global__ __launch_bounds__(kBlock) void k_pack_arena(const uint8_t* __restrict__ bytes,
                                                       const int32_t* __restrict__ offs,
                                                       const int32_t* __restrict__ perm, int64_t n,
                                                       const int32_t* __restrict__ lenstart,
                                                       const int64_t* __restrict__ gbase,
                                                       uint8_t* __restrict__ sarena,
                                                       uint16_t* __restrict__ slen, int lps_shift,
                                                       uint32_t* __restrict__ bitmap)
{
    __shared__ uint32_t seen[256];           // by byte value: not zero if present
    for (int k = threadIdx.x; k < 256; k += kBlock) seen[k] = 0;
    __syncthreads();
    const int lps = 1 << lps_shift;
    const int sub = threadIdx.x & (lps - 1);
    const int64_t total = offs[n];
    int64_t g = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> lps_shift;
    const int64_t gstep = ((int64_t)gridDim.x * kBlock) >> lps_shift;
    for (; g < n; g += gstep) {
        const int32_t id = perm[g];
        const int64_t a = offs[id];
        const int l = (int)(offs[id + 1] - a);
        uint4* dst = reinterpret_cast<uint4*>(sarena + gbase[l] + (g - lenstart[l]) * stride_of(l));
        if (sub == 0) slen[g] = (uint16_t)l;
        for (int q = sub; 16 * q < l; q += lps) {
            const int left = l - 16 * q;                   // bytes of the string from here on
            uint32_t w[4] = {0u, 0u, 0u, 0u};
            const uint8_t* src = bytes + a + 16 * q;
            if (a + 16 * q + 16 <= total) {
                const Unaligned16 v = *reinterpret_cast<const Unaligned16*>(src);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int in = left - 4 * k;           // bytes of the word inside the string
                    w[k] = in >= 4 ? v.w[k] : in > 0 ? v.w[k] & ((1u << (8 * in)) - 1u) : 0u;
                }
            } else {
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (k < left) w[k >> 2] |= (uint32_t)src[k] << (8 * (k & 3));
            }
            dst[q] = make_uint4(w[0], w[1], w[2], w[3]);
            if (bitmap) {
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const uint32_t byte = (w[k >> 2] >> ((k & 3) * 8)) & 255u;
                    if (k < left) seen[byte] = 1u;
                }
            }
        }
    }
    __syncthreads();
    if (bitmap && threadIdx.x < 8) {
        uint32_t m = 0;
        for (int k = 0; k < 32; ++k) m |= seen[32 * threadIdx.x + k] << k;
        if (m & ~__hip_atomic_load(&bitmap[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicOr(&bitmap[threadIdx.x], m);
    }
}

// ------------------------------------------------------------------------------------------
// Segment index
// ------------------------------------------------------------------------------------------

// One thread per (indexed string, slot), a string's slots together: emits (key, g) at a position
// grouped by (l, i) and ordered by g inside the group, so a stable sort by key keeps lists in
// ascending g.  Every block makes the symbol map from the bitmap of bytes present (bits and longest
// exact segment included, so the host need not wait for them here); the first writes it to `code`,
// and, with inl_base, where each length's inline copies begin.
__global__ __launch_bounds__(kBlock) void k_emit_segments(const uint8_t* __restrict__ sarena,
                                                          const uint16_t* __restrict__ slen,
                                                          const int32_t* __restrict__ lenstart,
                                                          const int64_t* __restrict__ gbase,
                                                          int tau, int64_t g_first,
                                                          int64_t g_count, Div div,
                                                          const uint32_t* __restrict__ bitmap,
                                                          uint16_t* __restrict__ code,
                                                          int64_t* __restrict__ inl_base,
                                                          uint64_t* __restrict__ keys,
                                                          uint32_t* __restrict__ vals)
{
    __shared__ uint16_t s_sym[256];
    const int T1 = tau + 1;
    uint32_t sigma = 0, rank = 0;
    for (int k = 0; k < 8; ++k) {
        const uint32_t word = bitmap[k];
        if (k == (int)(threadIdx.x >> 5))
            rank = (word >> (threadIdx.x & 31)) & 1u
                       ? sigma + (uint32_t)__popc(word & ((2u << (threadIdx.x & 31)) - 1u)) : 0u;
        sigma += (uint32_t)__popc(word);
    }
    s_sym[threadIdx.x] = (uint16_t)rank;
    const int bits = sigma < 2 ? 1 : 32 - __clz((int)sigma), exact_len = kHashBits / bits;
    if (blockIdx.x == 0) {
        code[threadIdx.x] = (uint16_t)rank;
        if (inl_base)
            for (int l = threadIdx.x; l < kLenTab; l += kBlock)
                inl_base[l] = l < T1 ? 0 : (gbase[l] - gbase[T1]) * T1 -
                                               (int64_t)(lenstart[l] - lenstart[T1]) * T1 * stride_of(l);
    }
    __syncthreads();
    const uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= (uint64_t)g_count * (uint32_t)T1) return;       // (fewer than 2^32 entries)
    const uint32_t at = (uint32_t)t / (uint32_t)T1;
    const int64_t g = g_first + at;
    const int i = (int)((uint32_t)t - at * (uint32_t)T1) + 1;
    const int l = slen[g];
    const Seg sg = partition_seg(l, i, tau, div);
    const int64_t ls = lenstart[l], nl = lenstart[l + 1] - ls;
    const uint8_t* s = sarena + gbase[l] + (g - ls) * stride_of(l);
    const uint64_t h = seg_code(s + sg.p - 1, sg.len, s_sym, bits, exact_len);
    const int64_t e = (ls - g_first) * T1 + (int64_t)(i - 1) * nl + (g - ls);
    keys[e] = make_key(l, i, tau, sg.len, h, exact_len);
    vals[e] = (uint32_t)g;
}

// Inline copies of the list members' strings: entry j of the sorted index (length l, read from
// its key's group) gets the bytes of string vals[j], in a slot of stride_of(l) bytes at
// inl + inl_base[l] + j * stride_of(l).  Entries of one length are contiguous in the sorted
// index (the group is the key's top field), so the copies of one list are contiguous too.
__global__ __launch_bounds__(kBlock) void k_gather_inline(
    const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals, int64_t E, int tau,
    const uint8_t* __restrict__ sarena, const int32_t* __restrict__ lenstart,
    const int64_t* __restrict__ gbase, const int64_t* __restrict__ inl_base,
    uint8_t* __restrict__ inl)
{
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= E) return;
    const int T1 = tau + 1;
    const int l = (int)((uint32_t)(keys[j] >> kHashBits) / (uint32_t)T1) + T1;
    const uint32_t g = vals[j];
    const int64_t st = stride_of(l);
    const uint4* src = reinterpret_cast<const uint4*>(sarena + gbase[l] +
                                                      (int64_t)(g - (uint32_t)lenstart[l]) * st);
    uint4* dst = reinterpret_cast<uint4*>(inl + inl_base[l] + j * st);
    for (int q = 0; q < (int)(st >> 4); ++q) dst[q] = src[q];
}

// One thread per list (and one more): its record, and the first and one-past-last list of each
// (l, i) group in bounds[g], bounds[ngroups + g] (zeroed by the caller): lists are in key order and
// the group is the key's top bits, so a group's lists are consecutive.
__global__ __launch_bounds__(kBlock) void k_list_records(const uint64_t* __restrict__ keys,
                                                         const uint32_t* __restrict__ runstart,
                                                         uint32_t nruns, uint32_t E,
                                                         uint32_t ngroups, uint4* __restrict__ recs,
                                                         uint32_t* __restrict__ bounds)
{
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    if (r > nruns) return;
    if (r == nruns) {
        recs[r] = make_uint4(~0u, ~0u, 0u, 0u);
        return;
    }
    const uint32_t start = runstart[r];
    const uint32_t end = r + 1 < nruns ? runstart[r + 1] : E;
    const uint64_t key = keys[start];
    recs[r] = make_uint4((uint32_t)key, (uint32_t)(key >> 32), start, end - start);
    const uint32_t g = (uint32_t)(key >> kHashBits);
    if (r == 0 || (uint32_t)(keys[start - 1] >> kHashBits) != g) bounds[g] = r;
    if (r + 1 == nruns || (uint32_t)(keys[end] >> kHashBits) != g) bounds[ngroups + g] = r + 1;
}

// entries of each group: the least power of two that is at least half its lists
__global__ __launch_bounds__(kBlock) void k_dir_words(const uint32_t* __restrict__ bounds,
                                                      uint32_t ngroups,
                                                      uint32_t* __restrict__ words)
{
    const uint32_t g = blockIdx.x * kBlock + threadIdx.x;
    if (g >= ngroups) return;
    const uint32_t need = (bounds[ngroups + g] - bounds[g] + 1) >> 1;
    uint32_t w = 1;
    while (w < need) w <<= 1;
    words[g] = w;
}

// One thread per list: the first list of a directory entry writes it, with the bits of all of
// them (one or two on average); entries without a list stay zero.  Lists in key order make both
// streaming writes: for 10^6 short strings at tau = 1 records, group sizes and directory take 31 us,
// where a hash table and a key filter filled by atomics took 242 (random 16-byte slots).
__global__ __launch_bounds__(kBlock) void k_dir_fill(const uint4* __restrict__ recs, uint32_t nruns,
                                                     const uint32_t* __restrict__ gdir,
                                                     uint2* __restrict__ dir)
{
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= nruns) return;
    auto key_of = [&](uint32_t q) {
        return *reinterpret_cast<const uint64_t*>(recs + q);   // a record starts with its key
    };
    const uint64_t key = key_of(r), g = key >> kHashBits;
    const uint32_t first = gdir[g];
    const uint32_t k = dir_bits(first, gdir[g + 1]);
    const uint32_t e = dir_entry(key, k);
    if (r > 0) {
        const uint64_t before = key_of(r - 1);
        if ((before >> kHashBits) == g && dir_entry(before, k) == e) return;
    }
    uint32_t map = 1u << dir_bit(key, k);
    for (uint32_t q = r + 1; q < nruns; ++q) {
        const uint64_t next = key_of(q);
        if ((next >> kHashBits) != g || dir_entry(next, k) != e) break;
        map |= 1u << dir_bit(next, k);
    }
    dir[first + e] = make_uint2(map, r);
}

// ------------------------------------------------------------------------------------------
// Probe: multi-match substring selection + list lookup (Sec. 4.2, Algorithm 2)
// ------------------------------------------------------------------------------------------

// One thread per (probe string x, probed length l, slot i), a wave over consecutive (l, i) pairs of
// one or a few probe strings.  The thread walks the window [bot_i, top_i] with a rolling code of
// x[p, l_i], looks each substring up, trims the list to the members visited before x (self-join,
// l == |x|), and appends non-empty lookups as hits.  Used for query batches (every string with a
// threshold of its own), in plain mode and where the autotuner asks for it.
constexpr int kProbeStep = 2;      // window positions a probe thread takes per step

// Members of the list [start, start + count) visited before gx (lists are in ascending g).
__device__ inline uint32_t members_before(const uint32_t* __restrict__ vals, uint32_t start,
                                          uint32_t count, uint32_t gx)
{
    uint32_t a = 0, b = count;
    while (a < b) {
        const uint32_t m = (a + b) >> 1;
        if (vals[start + m] < gx) a = m + 1; else b = m;
    }
    return a;
}

__global__ __launch_bounds__(kBlock) void k_probe(ProbeParams P, Div div)
{
    constexpr int kProbeStage = 2048;      // bytes of probe strings a wave stages in LDS
    __shared__ Hit s_hits[kWaves][kAppendCap];
    __shared__ uint4 s_xs[kWaves][kProbeStage / 16];
    __shared__ uint16_t s_sym[256];
    s_sym[threadIdx.x] = P.sym.code[threadIdx.x];
    __syncthreads();
    const int sym_bits = P.sym.bits, exact_len = P.sym.exact_len;
    const int lane = threadIdx.x & 63;
    WaveAppender<Hit, kAppendCap> app{s_hits[threadIdx.x >> 6], 0};
    const int T1 = P.tau + 1;
    const uint64_t nthreads = P.nx_dev ? (uint64_t)*P.nx_dev * (uint64_t)P.nl * (uint64_t)T1
                                       : P.threads;
    uint64_t my_sel = 0, my_cand = 0;
    // grid-stride over (probe string, length, slot) triples; the loop bound is block-uniform so
    // every lane takes part in the wave-level appends
    using LdsU8 = const __attribute__((address_space(3))) uint8_t*;
    const LdsU8 stage = (LdsU8)(s_xs[threadIdx.x >> 6]);
    const uint64_t per = (uint64_t)P.nl * T1;
    for (uint64_t t0 = (uint64_t)blockIdx.x * kBlock; t0 < nthreads;
         t0 += (uint64_t)gridDim.x * kBlock) {
        const uint64_t t = t0 + threadIdx.x;
        bool valid = t < nthreads;
        // the wave's threads cover consecutive probe strings; when they are of one length and
        // their padded bytes fit the stage, the wave copies them to LDS with 16-byte loads and
        // every byte of the window walk below is read from there (wave-uniform decision)
        const uint64_t tw = t0 + (threadIdx.x & ~63u);
        uint32_t g_first = 0;
        bool staged = false;
        const uint32_t gx_t = P.g_begin + (uint32_t)(t / per);
        const uint32_t r0 = (uint32_t)(t % per);
        if (tw < nthreads) {
            const uint64_t tl = min(tw + 63, nthreads - 1);
            g_first = P.g_begin + (uint32_t)(tw / per);
            const uint32_t g_last = P.g_begin + (uint32_t)(tl / per);
            const int n0 = P.x_slen[g_first];
            const int64_t bytes = (int64_t)(g_last - g_first + 1) * stride_of(n0);
            if (P.x_slen[g_last] == n0 && bytes <= kProbeStage) {
                staged = true;
                const uint4* src = reinterpret_cast<const uint4*>(
                    P.x_arena + P.x_gbase[n0] + (int64_t)(g_first - P.x_lenstart[n0]) * stride_of(n0));
                // the previous iteration's reads of the stage were issued before these writes,
                // and a wave's LDS requests complete in order
                for (int q = lane; q < (int)(bytes >> 4); q += 64) s_xs[threadIdx.x >> 6][q] = src[q];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
        }
        int n = 0, l = 0, i = 0, lo = 1, hi = 0, tau = P.tau;
        uint32_t gx = 0;
        Seg sg{1, 0};
        const uint8_t* x = nullptr;
        const uint4* recs = P.recs;
        const uint32_t* vals = P.vals;
        const uint2* dir = P.dir;
        const uint32_t* gdir = P.gdir;
        if (valid) {
            gx = gx_t;
            const uint32_t rem = P.order ? (uint32_t)P.order[r0] : r0;
            i = (int)(rem % T1) + 1;
            const int dl = (int)(rem / T1);
            n = P.x_slen[gx];
            Div dv = div;
            if (P.q_tau) {                       // mixed-tau batch: this probe string's own tau
                tau = P.q_tau[gx];
                const IndexRef ref = P.refs[tau];
                recs = ref.recs;
                vals = ref.vals;
                dir = ref.dir;
                gdir = ref.gdir;
                dv.d = (uint32_t)(tau + 1);
                dv.m = ref.div_m;
            }
            l = P.self ? n - dl : n - tau + dl;
            const bool in_window = i <= tau + 1 && dl <= (P.self ? tau : 2 * tau) && l >= tau + 1;
            // substrings selected for L_l^1 .. L_l^{tau+1}, whether or not strings of length l
            // exist (Algorithm 1 selects for every l in the length window): for multi-match
            // the Lemma 2 count, otherwise each slot's window size
            if (in_window && P.selection == 0 && i == 1) {
                const int d = n - l;
                my_sel += (uint64_t)((tau * tau - d * d) / 2 + tau + 1);
            }
            if (in_window) {
                sg = partition_seg(l, i, tau, dv);
                select_window(P.selection, n, l, tau, i, sg, &lo, &hi);
                if (P.selection != 0 && hi >= lo) my_sel += (uint64_t)(hi - lo + 1);
            }
            valid = in_window && (l >= P.ymin) && (l <= P.ymax) &&
                    (P.y_lenstart[l + 1] > P.y_lenstart[l]);
            if (valid)
                x = P.x_arena + P.x_gbase[n] + (int64_t)(gx - P.x_lenstart[n]) * stride_of(n);
        }
        const LdsU8 xs = stage + (int64_t)(gx - g_first) * stride_of(n);   // when staged
        auto rd = [&](int k) -> uint8_t { return staged ? xs[k] : x[k]; };
        uint64_t h = 0, top = 0;
        if (valid && lo <= hi) top = pow_hash(sg.len);   // HB^(len-1)
        // the (l, i) group's directory entries
        uint32_t dk = 0;
        if (valid && lo <= hi) {
            const uint32_t g = (uint32_t)((l - (tau + 1)) * (tau + 1) + (i - 1));
            const uint32_t first = gdir[g];
            dk = dir_bits(first, gdir[g + 1]);
            dir += first;
        }
        // the window has at most tau+1 positions for multi-match, more for the other methods;
        // the loop ends when no lane of the wave has a position left.  kProbeStep positions per
        // step: their bytes are read first, then their keys computed, then their directory
        // entries and the records these lead to read together, so a step waits on one round trip
        // per kind of read instead of one per position; hits are appended in position order.
        for (int s0 = 0;; s0 += kProbeStep) {
            if (__ballot(valid && lo + s0 <= hi) == 0) break;
            bool act[kProbeStep];
            int outb[kProbeStep], inb[kProbeStep];
#pragma unroll
            for (int u = 0; u < kProbeStep; ++u) {
                const int p = lo + s0 + u;
                act[u] = valid && p <= hi;
                outb[u] = 0;
                inb[u] = 0;
                if (act[u] && s0 + u > 0) {              // the bytes leaving and entering x[p, l_i]
                    outb[u] = rd(p - 2);
                    inb[u] = rd(p - 2 + sg.len);
                }
            }
            uint64_t key[kProbeStep];
#pragma unroll
            for (int u = 0; u < kProbeStep; ++u) {
                key[u] = 0;
                if (act[u]) {
                    if (s0 + u == 0) {
                        const int w0 = lo - 1;
                        h = 0;
                        if (sg.len <= exact_len)
                            for (int k = 0; k < sg.len; ++k) h = (h << sym_bits) | (uint64_t)s_sym[rd(w0 + k)];
                        else
                            for (int k = 0; k < sg.len; ++k) h = h * kHashBase + (uint64_t)rd(w0 + k) + 1ull;
                    } else {
                        h = roll_code(h, sg.len, (uint8_t)outb[u], (uint8_t)inb[u], top, s_sym,
                                      sym_bits, exact_len);
                    }
                    key[u] = make_key(l, i, tau, sg.len, h, exact_len);
                }
            }
            // one directory entry turns most absent segments away before a record is read
            uint2 de[kProbeStep];
#pragma unroll
            for (int u = 0; u < kProbeStep; ++u) {
                de[u] = make_uint2(0u, 0u);
                if (act[u]) de[u] = dir[dir_entry(key[u], dk)];
            }
            bool maybe[kProbeStep];
            uint4 rv[kProbeStep];
            uint32_t rn[kProbeStep];
#pragma unroll
            for (int u = 0; u < kProbeStep; ++u) {
                const uint32_t bit = dir_bit(key[u], dk);
                maybe[u] = (de[u].x >> bit) & 1u;
                rn[u] = de[u].y + (uint32_t)__popc(de[u].x & ((1u << bit) - 1u));
                rv[u] = make_uint4(0u, 0u, 0u, 0u);
                if (maybe[u]) rv[u] = recs[rn[u]];
            }
#pragma unroll
            for (int u = 0; u < kProbeStep; ++u) {
                uint32_t start = 0, count = 0;
                if (maybe[u]) {
                    const bool hit = find_record(recs, rn[u], key[u], rv[u], &start, &count);
                    if (hit && P.self && l == n) {
                        count = members_before(vals, start, count, gx);
                    }
                    if (!hit) count = 0;
                }
                const int p = lo + s0 + u;
                const bool found = act[u] && count > 0;
                Hit hh;
                hh.gx = gx; hh.start = start; hh.count = count;
                hh.meta = (uint32_t)(p - 1) | ((uint32_t)(i - 1) << 11) | ((uint32_t)l << 17);
                app.push(found, hh, P.hits, P.hit_cap, &P.counters[0]);
                if (found) my_cand += count;
            }
        }
    }
    block_flush(app, P.hits, P.hit_cap, &P.counters[0]);
    unsigned long long* line = stat_line(P.counters, P.shards);
    block_add(&line[1], my_cand);
    block_add(&line[2], my_sel);
}

// Pair-major probe.  A wave takes a tile of up to 64 probe strings of one length and, one after
// another, (length, slot) pairs: the partition, the window and the group's directory bounds are the
// same for its 64 lanes (scalar work), every lane walks a window of the same size, and consecutive
// waves look into the groups of a few lengths, whose directory and records stay in L2.  The strings
// are staged in lane slots of an odd number of words, so reads at one offset hit distinct banks.
// What bounds it is the random 8- and 16-byte reads of directory and records and, where most
// lookups hit, the atomic that reserves the places of a wave's HITS hits (6 ns each on one address):
// 512 from tau = 2 on in slots of up to 64 bytes, although a CU then holds three blocks and not six.
// Probe of 10^6 short strings at tau = 1 / 2 / 4: 0.37 / 0.64 / 2.62 ms string-major, here 0.096 /
// 0.30 / 2.17 with 256 hits and 0.108 / 0.22 / 1.14 with 512; 5x10^5 query lines at tau = 6 1.48 ms,
// 0.67 and 0.62, at tau = 8 2.04 and 1.46.
constexpr int kTileStep = 4;       // window positions in flight
constexpr uint32_t kStripes = 32;  // four an XCD: lengths differ in work

template <int MAXQ, int HITS>
__global__ __launch_bounds__(kBlock) void k_probe_tiles(ProbeParams P, Div div, ProbeTiles T)
{
    constexpr int SW = 4 * MAXQ + 1;               // words of a lane's slot
    __shared__ Hit s_hits[kWaves][HITS];
    __shared__ uint32_t s_x[kWaves][64 * SW];
    __shared__ uint16_t s_sym[256];
    s_sym[threadIdx.x] = P.sym.code[threadIdx.x];
    __syncthreads();
    const int sym_bits = P.sym.bits, exact_len = P.sym.exact_len;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    WaveAppender<Hit, HITS> app{s_hits[w], 0};
    uint32_t* slot = s_x[w] + lane * SW;
    using LdsU8 = const __attribute__((address_space(3))) uint8_t*;
    const LdsU8 xs = (LdsU8)slot;
    const int tau = P.tau, T1 = tau + 1;
    const uint32_t pairs = (uint32_t)P.nl * (uint32_t)T1;
    const uint32_t f0 = T.first[lane], f1 = T.first[64 + lane];
    uint64_t my_sel = 0, my_cand = 0;
    // Workgroups go to the XCDs round robin, and each XCD has an L2 of its own: an XCD takes every
    // eighth of kStripes stripes of consecutive tiles (strings of a few lengths, so of a few
    // groups), and its waves run through the stripe pair group by pair group.
    const uint32_t xcd = blockIdx.x & 7u, stripe = (T.tiles + kStripes - 1) / kStripes;
    const uint32_t units = kStripes / 8 * stripe * T.groups;          // of an XCD
    for (uint32_t u = (blockIdx.x >> 3) * kWaves + (uint32_t)w; u < units;
         u += (gridDim.x >> 3) * kWaves) {
        const uint32_t su = u / stripe, part = su % T.groups;
        const uint32_t tile = (su / T.groups * 8u + xcd) * stripe + u % stripe;
        if (tile >= T.tiles) continue;
        const int n = __popcll(__ballot(f0 <= tile)) + __popcll(__ballot(f1 <= tile)) - 1;
        const uint32_t n_first = (uint32_t)uniform_load(P.x_lenstart + n);
        const uint32_t g0 = n_first + (tile - T.first[n]) * 64u;
        const uint32_t cnt = min((uint32_t)uniform_load(P.x_lenstart + n + 1) - g0, 64u);
        const bool mine = (uint32_t)lane < cnt;
        const uint32_t gx = g0 + (uint32_t)lane;
        {
            const int nq = (n + 15) >> 4;
            const uint4* src = reinterpret_cast<const uint4*>(
                P.x_arena + uniform_load(P.x_gbase + n) + (int64_t)(g0 - n_first) * stride_of(n));
            // the previous unit's reads were issued before these writes (in order)
#pragma unroll
            for (int q = 0; q < MAXQ; ++q) {
                if (q < nq && mine) {
                    const uint4 v = src[lane * nq + q];
                    slot[4 * q] = v.x; slot[4 * q + 1] = v.y;
                    slot[4 * q + 2] = v.z; slot[4 * q + 3] = v.w;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        // the unit's pairs, 64 at a time: a lane finds one pair's window and directory block, then
        // the wave takes the pairs that have something to look up one by one
        for (uint32_t rb = part; rb < pairs; rb += 64 * T.groups) {
            const uint32_t rl = rb + (uint32_t)lane * T.groups;
            int v_lo = 1, v_hi = 0, v_len = 0, v_l = 0, v_i = 0;
            uint32_t v_first = 0, v_dk = 0;
            if (rl < pairs) {
                const int dl = (int)(rl / (uint32_t)T1);
                v_i = (int)(rl % (uint32_t)T1) + 1;
                v_l = P.self ? n - dl : n - tau + dl;
                if (v_l >= T1) {
                    // substrings selected whether or not strings of length l exist (Algorithm 1
                    // selects for every l in the length window): for multi-match the Lemma 2
                    // count, otherwise each slot's window size
                    const Seg sg = partition_seg(v_l, v_i, tau, div);
                    v_len = sg.len;
                    select_window(P.selection, n, v_l, tau, v_i, sg, &v_lo, &v_hi);
                    const int d = n - v_l;
                    if (P.selection != 0) my_sel += (uint64_t)cnt * (uint64_t)max(v_hi - v_lo + 1, 0);
                    else if (v_i == 1)
                        my_sel += (uint64_t)cnt * (uint64_t)((tau * tau - d * d) / 2 + tau + 1);
                    if (v_l >= P.ymin && v_l <= P.ymax &&
                        P.y_lenstart[v_l + 1] > P.y_lenstart[v_l]) {
                        const uint32_t grp = (uint32_t)((v_l - T1) * T1 + (v_i - 1));
                        v_first = P.gdir[grp];
                        v_dk = dir_bits(v_first, P.gdir[grp + 1]);
                    } else {
                        v_hi = 0;
                    }
                }
            }
            for (uint64_t todo = __ballot(v_lo <= v_hi); todo; todo &= todo - 1) {
                const int q = __ffsll((unsigned long long)todo) - 1;
                const int lo = __builtin_amdgcn_readlane(v_lo, q);
                const int hi = __builtin_amdgcn_readlane(v_hi, q);
                const int len = __builtin_amdgcn_readlane(v_len, q);
                const int l = __builtin_amdgcn_readlane(v_l, q);
                const int i = __builtin_amdgcn_readlane(v_i, q);
                const uint32_t dk = (uint32_t)__builtin_amdgcn_readlane((int)v_dk, q);
                const uint2* dir = P.dir + (uint32_t)__builtin_amdgcn_readlane((int)v_first, q);
                const uint64_t gkey = (uint64_t)((l - T1) * T1 + (i - 1)) << kHashBits;
                const bool exact = len <= exact_len;
                const uint64_t cmask = exact ? (1ull << (len * sym_bits)) - 1ull : 0ull;
                const uint64_t top = exact ? 0ull : pow_hash(len);
                uint64_t h = 0;
                if (exact)
                    for (int k = 0; k < len; ++k)
                        h = (h << sym_bits) | (uint64_t)s_sym[xs[lo - 1 + k]];
                else
                    for (int k = 0; k < len; ++k)
                        h = h * kHashBase + (uint64_t)xs[lo - 1 + k] + 1ull;
                for (int p0 = lo; p0 <= hi; p0 += kTileStep) {
                    uint64_t key[kTileStep];
                    uint2 de[kTileStep];
#pragma unroll
                    for (int v = 0; v < kTileStep; ++v) {
                        const int p = p0 + v;
                        de[v] = make_uint2(0u, 0u);
                        key[v] = 0;
                        if (p > hi) continue;
                        if (p > lo) {
                            if (exact)
                                h = ((h << sym_bits) | (uint64_t)s_sym[xs[p - 2 + len]]) & cmask;
                            else
                                h = roll_hash(h, xs[p - 2], xs[p - 2 + len], top);
                        }
                        key[v] = gkey | spread_code(len, h, exact_len);
                        if (mine) de[v] = dir[dir_entry(key[v], dk)];
                    }
                    uint4 rv[kTileStep];
#pragma unroll
                    for (int v = 0; v < kTileStep; ++v) {
                        const uint32_t bit = dir_bit(key[v], dk);
                        rv[v] = make_uint4(0u, 0u, 0u, 0u);
                        if ((de[v].x >> bit) & 1u) {
                            de[v].y += (uint32_t)__popc(de[v].x & ((1u << bit) - 1u));
                            rv[v] = P.recs[de[v].y];
                        } else {
                            de[v].x = 0;
                        }
                    }
#pragma unroll
                    for (int v = 0; v < kTileStep; ++v) {
                        if (__ballot(de[v].x != 0) == 0) continue;
                        uint32_t start = 0, count = 0;
                        if (de[v].x != 0) {
                            const bool hit =
                                find_record(P.recs, de[v].y, key[v], rv[v], &start, &count);
                            if (!hit) count = 0;
                            else if (P.self && l == n)
                                count = members_before(P.vals, start, count, gx);
                        }
                        Hit hh;
                        hh.gx = gx; hh.start = start; hh.count = count;
                        hh.meta = (uint32_t)(p0 + v - 1) | ((uint32_t)(i - 1) << 11) |
                                  ((uint32_t)l << 17);
                        app.push(count > 0, hh, P.hits, P.hit_cap, &P.counters[0]);
                        my_cand += count;
                    }
                }
            }
        }
    }
    block_flush(app, P.hits, P.hit_cap, &P.counters[0]);
    unsigned long long* line = stat_line(P.counters, P.shards);
    block_add(&line[1], my_cand);
    block_add(&line[2], my_sel);
}

// Multi-match probe of long strings, a block per string.  Hashing every window's first segment byte
// by byte and rolling on made a chain of thousands of multiplications per lane (the first segments
// alone are nl * n bytes a string), and lanes with small windows waited for those with large ones.
// Here the block computes the polynomial hashes of all prefixes once (a scan over the bytes:
// H(ab) = H(a) B^|b| + H(b)), so any segment's hash is H[p + len] - H[p] B^len; notes every pair's
// directory block in LDS; and takes the windows' positions from one list, 256 at a time.  The next
// string's bytes are read meanwhile.  Vector issue bounds it (64-bit multiplications).  10^5 long
// strings at tau = 16: 1.98 -> 1.20 ms.  NMAX: the longest string (LDS).
template <int NMAX>
__global__ __launch_bounds__(kBlock) void k_probe_long(ProbeParams P, Div div, ProbeItems I,
                                                       uint32_t g_first, uint32_t g_end)
{
    constexpr int CAP = 64;                        // hits are rare
    constexpr int U = 4;                           // positions a thread has in flight
    __shared__ Hit s_hits[kWaves][CAP];
    __shared__ uint64_t s_pre[NMAX];               // hashes of the prefixes of 0 .. NMAX - 1 bytes
    __shared__ uint4 s_b4[NMAX / 16];              // the string's bytes
    __shared__ uint32_t s_first[kItemPairs], s_grp[kItemPairs], s_pair[kItemPairs];
    __shared__ uint64_t s_wave[kWaves], s_pow[4];
    __shared__ uint16_t s_sym[256];
    s_sym[threadIdx.x] = P.sym.code[threadIdx.x];
    const uint8_t* s_b = reinterpret_cast<const uint8_t*>(s_b4);
    const int sym_bits = P.sym.bits, exact_len = P.sym.exact_len;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    WaveAppender<Hit, CAP> app{s_hits[w], 0};
    const int tau = P.tau, T1 = tau + 1;
    const uint32_t pairs = (uint32_t)P.nl * (uint32_t)T1;
    uint64_t my_sel = 0, my_cand = 0;
    // a string's length and the thread's 16 bytes of it
    auto fetch = [&](uint32_t gx, int& n, uint4& v) {
        n = __builtin_amdgcn_readfirstlane((int)P.x_slen[gx]);
        const uint4* src = reinterpret_cast<const uint4*>(
            P.x_arena + uniform_load(P.x_gbase + n) +
            (int64_t)(gx - (uint32_t)uniform_load(P.x_lenstart + n)) * stride_of(n));
        if ((int)threadIdx.x < (n + 15) / 16) v = src[threadIdx.x];
    };
    uint32_t gx = g_first + blockIdx.x;
    int n_next = 0;
    uint4 v_next = make_uint4(0u, 0u, 0u, 0u);
    if (gx < g_end) fetch(gx, n_next, v_next);
    for (; gx < g_end; gx += gridDim.x) {
        const int n = n_next;
        __syncthreads();                           // the previous string's reads are done
        if ((int)threadIdx.x < (n + 15) / 16) s_b4[threadIdx.x] = v_next;
        if (gx + gridDim.x < g_end) fetch(gx + gridDim.x, n_next, v_next);
        // segments of the probed lengths have at most four lengths, from qlo on
        const int qlo = div(max(n - tau, T1));
        if (threadIdx.x < 4) s_pow[threadIdx.x] = pow_hash(qlo + (int)threadIdx.x + 1);
        __syncthreads();
        // prefix hashes: thread t takes bytes [t * c, t * c + c) (bytes past the end count as
        // nothing: they only enter prefixes that are never read)
        const int c = (n + kBlock - 1) / kBlock;
        const int b0 = (int)threadIdx.x * c;
        uint64_t v = 0, bc = 1;
        for (int k = 0; k < c; ++k) {
            v = v * kHashBase + (b0 + k < n ? (uint64_t)s_b[b0 + k] + 1ull : 0ull);
            bc *= kHashBase;
        }
        uint64_t mul = bc, bl = 1;                 // B^(bytes a lane's v covers), B^(lane * c)
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            const uint64_t before = __shfl_up(v, 1 << b, 64);
            if (lane >= 1 << b) v += before * mul;
            if ((lane >> b) & 1) bl *= mul;
            mul *= mul;
        }
        if (lane == 63) s_wave[w] = v;
        uint64_t run = __shfl_up(v, 1, 64);
        if (lane == 0) run = 0;
        __syncthreads();
        uint64_t carry = 0;                        // the waves before: 64 * c bytes each
        for (int k = 0; k < w; ++k) carry = carry * mul + s_wave[k];
        run += carry * bl;
        if (threadIdx.x == 0) s_pre[0] = 0;
        for (int k = 0; k < c && b0 + k < n; ++k) {
            run = run * kHashBase + (uint64_t)s_b[b0 + k] + 1ull;
            s_pre[b0 + k + 1] = run;
        }
        for (int ch = 0; ch < I.chunks; ++ch) {
            const uint32_t rbase = (uint32_t)ch * kItemPairs;
            if (ch > 0) __syncthreads();           // the previous chunk's reads are done
            for (uint32_t q = threadIdx.x; q < (uint32_t)kItemPairs && rbase + q < pairs; q += kBlock) {
                const uint32_t r = rbase + q;
                const int dl = (int)(r / (uint32_t)T1);
                const int i = (int)(r % (uint32_t)T1) + 1;
                const int l = P.self ? n - dl : n - tau + dl;
                uint32_t info = 0;                 // no segment: nothing to look up
                if (l >= T1) {
                    // the Lemma 2 count, whether or not strings of length l exist (Algorithm 1
                    // selects for every l in the length window)
                    const int d = n - l;
                    if (i == 1) my_sel += (uint64_t)((tau * tau - d * d) / 2 + tau + 1);
                    if (l >= P.ymin && l <= P.ymax && P.y_lenstart[l + 1] > P.y_lenstart[l]) {
                        const Seg sg = partition_seg(l, i, tau, div);
                        const int rr = tau + 1 - i;
                        const int p0 = max(sg.p - (i - 1), sg.p + d - rr);   // unclipped start
                        const uint32_t grp = (uint32_t)((l - T1) * T1 + (i - 1));
                        const uint32_t first = P.gdir[grp];
                        s_first[q] = first;
                        s_grp[q] = grp;
                        info = (uint32_t)sg.len | dir_bits(first, P.gdir[grp + 1]) << 11 |
                               (uint32_t)(p0 + 128) << 16;
                    }
                }
                s_pair[q] = info;
            }
            __syncthreads();
            const uint32_t i0 = uniform_load(I.chunk + ch), i1 = uniform_load(I.chunk + ch + 1);
            for (uint32_t base = i0 + (uint32_t)w * 64u; base < i1; base += kBlock * U) {
                uint32_t q[U];
                int p[U];
                uint64_t key[U];
                uint2 de[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t it = base + (uint32_t)(u * kBlock + lane);
                    q[u] = it < i1 ? I.items[it] : ~0u;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    p[u] = 0;
                    key[u] = 0;
                    de[u] = make_uint2(0u, 0u);
                    if (q[u] == ~0u) continue;
                    const int s = (int)(q[u] & 255u);
                    q[u] = (q[u] >> 8) - rbase;
                    const uint32_t info = s_pair[q[u]];
                    const int len = (int)(info & 2047u);
                    const int at = (int)(info >> 16) - 128 + s;
                    if (len == 0 || at < 1 || at > n - len + 1) continue;
                    p[u] = at;
                    uint64_t h = 0;
                    if (len <= exact_len)
                        for (int k = 0; k < len; ++k)
                            h = (h << sym_bits) | (uint64_t)s_sym[s_b[at - 1 + k]];
                    else
                        h = s_pre[at - 1 + len] - s_pre[at - 1] * s_pow[len - qlo];
                    key[u] = (uint64_t)s_grp[q[u]] << kHashBits | spread_code(len, h, exact_len);
                    const uint32_t k = (info >> 11) & 31u;
                    de[u] = P.dir[s_first[q[u]] + dir_entry(key[u], k)];
                    p[u] |= (int)(dir_bit(key[u], k) << 16);
                }
                uint4 rv[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t bit = (uint32_t)p[u] >> 16;
                    rv[u] = make_uint4(0u, 0u, 0u, 0u);
                    if ((de[u].x >> bit) & 1u) {
                        de[u].y += (uint32_t)__popc(de[u].x & ((1u << bit) - 1u));
                        rv[u] = P.recs[de[u].y];
                    } else {
                        de[u].x = 0;
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (__ballot(de[u].x != 0) == 0) continue;
                    uint32_t start = 0, count = 0;
                    Hit hh{};
                    if (de[u].x != 0) {
                        const bool hit = find_record(P.recs, de[u].y, key[u], rv[u], &start, &count);
                        const uint32_t r = rbase + q[u];
                        const int dl = (int)(r / (uint32_t)T1), i0m = (int)(r % (uint32_t)T1);
                        const int l = P.self ? n - dl : n - tau + dl;
                        if (!hit) count = 0;
                        else if (P.self && l == n) count = members_before(P.vals, start, count, gx);
                        hh.gx = gx; hh.start = start; hh.count = count;
                        hh.meta = ((uint32_t)p[u] & 0xffffu) - 1u | (uint32_t)i0m << 11 |
                                  (uint32_t)l << 17;
                    }
                    app.push(count > 0, hh, P.hits, P.hit_cap, &P.counters[0]);
                    my_cand += count;
                }
            }
        }
    }
    block_flush(app, P.hits, P.hit_cap, &P.counters[0]);
    unsigned long long* line = stat_line(P.counters, P.shards);
    block_add(&line[1], my_cand);
    block_add(&line[2], my_sel);
}

// ------------------------------------------------------------------------------------------
// Verify: extension-based verification (Sec. 5.2, Algorithm 3), lane per candidate, candidates
// distributed over lanes by a load-balanced search over the hits' prefix sums.
// ------------------------------------------------------------------------------------------

constexpr int kVerifyChunk = 1024;

template <int MAXW>
__global__ __launch_bounds__(kBlock) void k_verify(VerifyParams V, Div div)
{
    __shared__ unsigned long long sP[kVerifyChunk + 1];
    __shared__ uint64_t s_h0;
    const int lane = threadIdx.x & 63;
    uint64_t my_cells = 0, my_miss = 0;
    const uint64_t nchunks = (V.ncand + kVerifyChunk - 1) / kVerifyChunk;
    for (uint64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        const uint64_t c0 = ch * kVerifyChunk;
        const uint64_t c1 = (c0 + kVerifyChunk < V.ncand) ? c0 + kVerifyChunk : V.ncand;
        if (threadIdx.x == 0) {
            uint64_t a = 0, b = V.nhits - 1;      // largest h with prefix[h] <= c0
            while (a < b) {
                uint64_t m = (a + b + 1) >> 1;
                if (V.prefix[m] <= c0) a = m; else b = m - 1;
            }
            s_h0 = a;
        }
        __syncthreads();
        const uint64_t h0 = s_h0;
        for (int k = threadIdx.x; k <= kVerifyChunk; k += kBlock)
            sP[k] = (h0 + k <= V.nhits) ? V.prefix[h0 + k] : ~0ull;
        __syncthreads();
        for (uint64_t c = c0 + threadIdx.x; c - c0 < (uint64_t)kVerifyChunk; c += kBlock) {
            bool pass = false;
            uint32_t gx = 0, gy = 0;
            if (c < c1) {
                int a = 0, b = kVerifyChunk;
                while (a < b) {
                    int m = (a + b + 1) >> 1;
                    if (sP[m] <= c) a = m; else b = m - 1;
                }
                const Hit hit = V.hits[h0 + a];
                const uint64_t mem = c - sP[a];
                gx = hit.gx;
                int tau = V.tau;
                const uint32_t* vals = V.vals;
                Div dv = div;
                if (V.q_tau) {
                    tau = V.q_tau[gx];
                    vals = V.refs[tau].vals;
                    dv.d = (uint32_t)(tau + 1);
                    dv.m = V.refs[tau].div_m;
                }
                gy = vals[hit.start + mem];
                const int p = (int)(hit.meta & 2047u) + 1;
                const int i = (int)((hit.meta >> 11) & 63u) + 1;
                const int l = (int)(hit.meta >> 17);
                const int n = V.x_slen[gx];
                const uint8_t* x = V.x_arena + V.x_gbase[n] +
                                   (int64_t)(gx - V.x_lenstart[n]) * stride_of(n);
                const uint8_t* y = V.y_arena + V.y_gbase[l] +
                                   (int64_t)(gy - V.y_lenstart[l]) * stride_of(l);
                const Seg sg = partition_seg(l, i, tau, dv);
                bool same = true;
                if (sg.len > V.exact_len)
                    for (int k = 0; k < sg.len; ++k) same &= (x[p - 1 + k] == y[sg.p - 1 + k]);
                if (!same) {
                    my_miss += 1;
                } else {
                    int cl = 0;
                    const int tl = i - 1, tr = tau + 1 - i;
                    int dl = vsp_global<MAXW>(y, sg.p - 1, x, p - 1, tl, &cl);
                    my_cells += cl;
                    if (dl <= tl) {
                        int cr = 0;
                        const int ry = sg.p - 1 + sg.len, rx = p - 1 + sg.len;
                        int dr = vsp_global<MAXW>(y + ry, l - ry, x + rx, n - rx, tr, &cr);
                        my_cells += cr;
                        pass = dr <= tr;
                    }
                }
            }
            uint64_t pm = __ballot(pass);
            if (pm) {
                int leader = __ffsll((unsigned long long)pm) - 1;
                unsigned long long base = 0;
                if (lane == leader) base = atomicAdd(&V.counters[3], (unsigned long long)__popcll(pm));
                base = __shfl(base, leader, 64);
                if (pass) {
                    uint64_t idx = base + (uint64_t)__popcll(pm & lanemask_lt());
                    if (idx < V.out_cap) V.out[idx] = ((uint64_t)gx << 32) | gy;
                }
            }
        }
        __syncthreads();
    }
    unsigned long long* line = stat_line(V.counters, V.shards);
    block_add(&line[4], my_cells);
    block_add(&line[5], my_miss);
}

// ------------------------------------------------------------------------------------------
// Batched verification.  Hits are bucketed by slot i, so the candidates of a wave almost always
// share (tau_l, tau_r) = (i - 1, tau + 1 - i) and run band DPs of exactly that width.  Each wave
// walks its own chunks of 64 x kWaveRounds consecutive candidates; the hit of each lane is found
// from the hits' end offsets with one OR-reduced boundary mask per 64 candidates.
// ------------------------------------------------------------------------------------------

constexpr int kWaveRounds = kBatchedRoundsMax;

// Bucket of a hit: small lists, then big ones (from 64 * kLenClasses on), each by the length
// class of the list's strings and then by slot
__device__ inline uint32_t hit_bucket(const Hit& v, uint32_t big)
{
    const uint32_t slot = (v.meta >> 11) & 63u;
    const uint32_t cls = (uint32_t)len_class((int)(v.meta >> 17));
    return (v.count < big ? 0u : 64u * (uint32_t)kLenClasses) + 64u * cls + slot;
}

// Bucketing of the hits in two passes without global atomics: bb[b * G + blk] = hits of
// bucket b that block blk meets in its grid-stride walk (G blocks, kBuckets buckets); after an
// exclusive scan of bb (bucket-major), the scatter pass walks the same hits in the same order
// and places each at its block's offset in its bucket plus a rank from LDS counters.  The
// regions come out in bucket order; order inside a region changes nothing downstream (the
// result is sorted).
__global__ __launch_bounds__(kBlock) void k_slot_hist(const Hit* __restrict__ hits,
                                                      const unsigned long long* __restrict__ nh_dev,
                                                      uint32_t big, uint32_t* __restrict__ bb)
{
    __shared__ uint32_t h[kHitBuckets];
    for (int b = threadIdx.x; b < kHitBuckets; b += kBlock) h[b] = 0;
    __syncthreads();
    const uint64_t nh = *nh_dev;
    for (uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x; k < nh;
         k += (uint64_t)gridDim.x * kBlock)
        atomicAdd(&h[hit_bucket(hits[k], big)], 1u);
    __syncthreads();
    for (int b = threadIdx.x; b < kHitBuckets; b += kBlock)
        bb[(uint64_t)b * gridDim.x + blockIdx.x] = h[b];
}

__global__ __launch_bounds__(kBlock) void k_slot_scatter(const Hit* __restrict__ hits,
                                                         const unsigned long long* __restrict__ nh_dev,
                                                         uint32_t big,
                                                         const uint32_t* __restrict__ bb_off,
                                                         Hit* __restrict__ out)
{
    __shared__ uint32_t run[kHitBuckets], cnt[kHitBuckets];
    for (int b = threadIdx.x; b < kHitBuckets; b += kBlock)
        run[b] = bb_off[(uint64_t)b * gridDim.x + blockIdx.x];
    const uint64_t nh = *nh_dev;
    for (uint64_t k0 = (uint64_t)blockIdx.x * kBlock; k0 < nh; k0 += (uint64_t)gridDim.x * kBlock) {
        for (int b = threadIdx.x; b < kHitBuckets; b += kBlock) cnt[b] = 0;
        __syncthreads();
        const uint64_t k = k0 + threadIdx.x;
        Hit v{};
        uint32_t sl = 0, rank = 0;
        if (k < nh) {
            v = hits[k];
            sl = hit_bucket(v, big);
            rank = atomicAdd(&cnt[sl], 1u);
        }
        __syncthreads();
        if (k < nh) out[run[sl] + rank] = v;
        __syncthreads();
        for (int b = threadIdx.x; b < kHitBuckets; b += kBlock) run[b] += cnt[b];
    }
}

// first[ch] = the hit containing candidate ch * chunk (largest h with prefix[h] <= it)
__global__ __launch_bounds__(kBlock) void k_chunk_starts(const unsigned long long* __restrict__ prefix,
                                                         uint64_t nhits, uint64_t nchunks,
                                                         uint64_t chunk,
                                                         uint32_t* __restrict__ first)
{
    const uint64_t ch = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (ch >= nchunks) return;
    const unsigned long long c0 = ch * chunk;
    uint64_t a = 0, b = nhits - 1;
    while (a < b) {
        const uint64_t m = (a + b + 1) >> 1;
        if (prefix[m] <= c0) a = m; else b = m - 1;
    }
    first[ch] = (uint32_t)a;
}

__device__ inline uint64_t wave_or64(uint64_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v |= __shfl_xor(v, d, 64);
    return v;
}

// VerifyStringPair with the band width fixed at compile time when the threshold is the same on
// every active lane of the wave (t <= 8), else the generic width class GMAXW.
template <int GMAXW, typename P>
__device__ inline int vsp_dispatch(P r, int lr, P s, int ls, int t, int* cells)
{
    const int t0 = __builtin_amdgcn_readfirstlane(t);
    if (t0 <= 8 && __ballot(t != t0) == 0) {
        switch (t0) {
        case 0: return vsp_fast<1>(r, lr, s, ls, t, cells);
        case 1: return vsp_fast<2>(r, lr, s, ls, t, cells);
        case 2: return vsp_fast<3>(r, lr, s, ls, t, cells);
        case 3: return vsp_fast<4>(r, lr, s, ls, t, cells);
        case 4: return vsp_fast<5>(r, lr, s, ls, t, cells);
        case 5: return vsp_fast<6>(r, lr, s, ls, t, cells);
        case 6: return vsp_fast<7>(r, lr, s, ls, t, cells);
        case 7: return vsp_fast<8>(r, lr, s, ls, t, cells);
        default: return vsp_fast<9>(r, lr, s, ls, t, cells);
        }
    }
    // wider uniform thresholds (long strings, tau up to 32): a class of at most 3 extra columns
    if constexpr (GMAXW > 9 && GMAXW <= 33) {
        if (__ballot(t != t0) == 0) {
            if (t0 + 1 <= 13) return vsp_fast<13>(r, lr, s, ls, t, cells);
            if constexpr (GMAXW > 17) {
                if (t0 + 1 <= 17) return vsp_fast<17>(r, lr, s, ls, t, cells);
                if (t0 + 1 <= 21) return vsp_fast<21>(r, lr, s, ls, t, cells);
                if (t0 + 1 <= 25) return vsp_fast<25>(r, lr, s, ls, t, cells);
                if (t0 + 1 <= 29) return vsp_fast<29>(r, lr, s, ls, t, cells);
            }
        }
    }
    return vsp_fast<GMAXW>(r, lr, s, ls, t, cells);
}

// STG: every lane copies its candidate's two strings into LDS slots of its own first (probe
// string x up to kStgX - 4 bytes, indexed string y up to kStgY - 4), so the band DP reads LDS
// instead of global memory byte by byte.  Launched for indexed strings of at most 48 bytes and
// tau <= 8: a hit pairs x with lists of lengths within tau of |x|, so |x| <= 56.  STG 2 is the
// form for indexed strings of at most 40 bytes (|x| <= 48) with 52- and 44-byte slots and a
// 128-pair buffer: 28 KB per block, 5 blocks per CU, registers held to 96 (a 104-byte spill);
// it is taken for tau 6..8, where the fifth wave paid (the self-join of 5x10^5 medium strings:
// 22.1 -> 21.5 ms at tau = 8), not below (2% slower at tau 2 and 4 on short strings).
constexpr int kStgX = 60, kStgY = 52;     // slot strides: odd word counts, conflict-free

// With STG the LDS slots allow 4 blocks per CU; the register budget is held to match
// (128 VGPRs, no spills), so 4 waves per SIMD hide the candidates' dependent loads.  The
// unstaged 9-wide form is held to 128 VGPRs too (it would take 135, 3 waves per SIMD; the
// budget costs an 8-byte spill and gains a wave: the self-join of 5x10^5 medium strings at
// tau 2..8 measured 37.5 -> 36.0 ms); the wider bands keep their registers.
template <int GMAXW, int STG>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(STG == 2 ? 5 : (STG || GMAXW <= 9) ? 4 : 1))) void k_verify_batched(VerifyParams V, Div div,
                                                           const uint32_t* __restrict__ first,
                                                           uint64_t nchunks)
{
    // slot strides and pair buffer: STG 2 the smaller ones (5 blocks per CU in LDS)
    constexpr int SX = STG == 2 ? 52 : kStgX, SY = STG == 2 ? 44 : kStgY;
    constexpr int ACAP = STG == 2 ? 128 : kAppendCap;
    __shared__ uint64_t s_acc[kWaves][ACAP];
    __shared__ uint32_t s_str[kWaves][STG ? 64 * (SX + SY) / 4 : 1];
    WaveAppender<uint64_t, ACAP> acc{s_acc[threadIdx.x >> 6], 0};
    const int lane = threadIdx.x & 63;
    using LdsBytes = const __attribute__((address_space(3))) uint8_t*;
    __attribute__((address_space(3))) uint32_t* xsw =
        (__attribute__((address_space(3))) uint32_t*)(s_str[threadIdx.x >> 6]) + lane * (SX / 4);
    __attribute__((address_space(3))) uint32_t* ysw =
        (__attribute__((address_space(3))) uint32_t*)(s_str[threadIdx.x >> 6]) + 64 * (SX / 4) +
        lane * (SY / 4);
    const uint64_t wave = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const uint64_t nwaves = ((uint64_t)gridDim.x * kBlock) >> 6;
    uint64_t my_cells = 0, my_miss = 0;
    const uint64_t le_mask = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    const uint64_t nhits = V.dev_counts ? V.dev_counts[0] : V.nhits;
    const uint64_t ncand = V.dev_counts ? V.dev_counts[1] : V.ncand;
    const uint64_t nch = V.dev_counts ? V.dev_counts[2] : nchunks;
    const uint64_t chunk = 64ull * (V.dev_counts ? V.dev_counts[4] : (uint64_t)V.wave_rounds);
    for (uint64_t ch = wave; ch < nch; ch += nwaves) {
        const uint64_t c0 = ch * chunk;
        const uint64_t cend = (c0 + chunk < ncand) ? c0 + chunk : ncand;
        uint64_t h = first[ch];
        unsigned long long hstart = V.prefix[h];
        for (uint64_t g0 = c0; g0 < cend; g0 += 64) {
            // end offsets of hits h .. h + 63; a boundary at relative position r means the
            // candidates from r on belong to later hits
            const uint64_t hk = h + (uint64_t)lane;
            const unsigned long long bk = (hk < nhits) ? V.prefix[hk + 1] : ~0ull;
            const uint64_t rel = bk - g0;                      // >= 1
            const uint64_t M = wave_or64(rel < 64 ? (1ull << rel) : 0ull);
            const int off = __popcll(M & le_mask);
            const unsigned long long bprev = __shfl(bk, off > 0 ? off - 1 : 0, 64);
            const unsigned long long hs = (off == 0) ? hstart : bprev;
            const uint64_t c = g0 + (uint64_t)lane;
            bool pass = false;
            uint32_t gx = 0, gy = 0;
            if (c < cend) {
                const Hit hit = V.hits[h + (uint64_t)off];
                const uint64_t mem = c - hs;
                gx = hit.gx;
                int tau = V.tau;
                const uint32_t* vals = V.vals;
                Div dv = div;
                if (V.q_tau) {
                    tau = V.q_tau[gx];
                    vals = V.refs[tau].vals;
                    dv.d = (uint32_t)(tau + 1);
                    dv.m = V.refs[tau].div_m;
                }
                gy = vals[hit.start + mem];
                const int p = (int)(hit.meta & 2047u) + 1;
                const int i = (int)((hit.meta >> 11) & 63u) + 1;
                const int l = (int)(hit.meta >> 17);
                const int n = V.x_slen[gx];
                const uint8_t* x = V.x_arena + V.x_gbase[n] +
                                   (int64_t)(gx - V.x_lenstart[n]) * stride_of(n);
                const uint8_t* y = V.y_arena + V.y_gbase[l] +
                                   (int64_t)(gy - V.y_lenstart[l]) * stride_of(l);
                const Seg sg = partition_seg(l, i, tau, dv);
                auto verify = [&](auto xp, auto yp) {
                    bool same = true;
                    if (sg.len > V.exact_len)
                        for (int k = 0; k < sg.len; ++k) same &= (xp[p - 1 + k] == yp[sg.p - 1 + k]);
                    if (!same) {
                        my_miss += 1;
                        return;
                    }
                    int cl = 0;
                    const int tl = i - 1, tr = tau + 1 - i;
                    const int dl = vsp_dispatch<GMAXW>(yp, sg.p - 1, xp, p - 1, tl, &cl);
                    my_cells += cl;
                    if (dl <= tl) {
                        int cr = 0;
                        const int ry = sg.p - 1 + sg.len, rx = p - 1 + sg.len;
                        const int dr =
                            vsp_dispatch<GMAXW>(yp + ry, l - ry, xp + rx, n - rx, tr, &cr);
                        my_cells += cr;
                        pass = dr <= tr;
                    }
                };
                if constexpr (STG > 0) {
                    const uint4* xq = reinterpret_cast<const uint4*>(x);
                    const uint4* yq = reinterpret_cast<const uint4*>(y);
#pragma unroll
                    for (int q = 0; q < (SX + 15) / 16; ++q) {
                        if (q * 16 < n) {
                            const uint4 v = xq[q];
                            if (4 * q < SX / 4) xsw[4 * q] = v.x;
                            if (4 * q + 1 < SX / 4) xsw[4 * q + 1] = v.y;
                            if (4 * q + 2 < SX / 4) xsw[4 * q + 2] = v.z;
                            if (4 * q + 3 < SX / 4) xsw[4 * q + 3] = v.w;
                        }
                    }
#pragma unroll
                    for (int q = 0; q < (SY + 15) / 16; ++q) {
                        if (q * 16 < l) {
                            const uint4 v = yq[q];
                            if (4 * q < SY / 4) ysw[4 * q] = v.x;
                            if (4 * q + 1 < SY / 4) ysw[4 * q + 1] = v.y;
                            if (4 * q + 2 < SY / 4) ysw[4 * q + 2] = v.z;
                            if (4 * q + 3 < SY / 4) ysw[4 * q + 3] = v.w;
                        }
                    }
                    verify((LdsBytes)(xsw), (LdsBytes)(ysw));
                } else {
                    verify(x, y);
                }
            }
            acc.push(pass, ((uint64_t)gx << 32) | gy, V.out, V.out_cap, &V.counters[3]);
            // the hit containing candidate g0 + 64 starts the next group
            const uint64_t nb = __ballot(rel <= 64);
            const int adv = __popcll(nb);
            if (adv > 0) {
                hstart = __shfl(bk, adv - 1, 64);
                h += (uint64_t)adv;
            }
        }
    }
    block_flush(acc, V.out, V.out_cap, &V.counters[3]);
    unsigned long long* line = stat_line(V.counters, V.shards);
    block_add(&line[4], my_cells);
    block_add(&line[5], my_miss);
}

// ------------------------------------------------------------------------------------------
// List-segment verification: a wave verifies up to 64 members of one inverted list against
// the same probe substring, so the probe string, the partition and both band geometries are
// wave-uniform and only the indexed string differs per lane.  Used for lists with at least
// kBigList candidates; smaller lists go through k_verify_batched.
// ------------------------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_seg_counts(const Hit* __restrict__ hits, uint64_t nbig,
                                                       uint32_t members, uint32_t* __restrict__ segs)
{
    const uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k < nbig) segs[k] = (hits[k].count + members - 1u) / members;
}

// first[ch] = the list holding segment ch * chunk (largest h with segp[h] <= it)
__global__ __launch_bounds__(kBlock) void k_seg_chunk_starts(const uint32_t* __restrict__ segp,
                                                             uint64_t nbig, uint64_t nchunks,
                                                             uint32_t chunk,
                                                             uint32_t* __restrict__ first)
{
    const uint64_t ch = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (ch >= nchunks) return;
    const uint64_t s0 = ch * chunk;
    uint64_t a = 0, b = nbig - 1;
    while (a < b) {
        const uint64_t m = (a + b + 1) >> 1;
        if (segp[m] <= s0) a = m; else b = m - 1;
    }
    first[ch] = (uint32_t)a;
}

using LdsInts = const __attribute__((address_space(3))) int*;

template <int MAXW, int NC, int TS, typename LaneChars>
__device__ inline void vsp_seg_any(bool yrows, LdsChars U, int lu, const LaneChars (&V)[NC],
                                   int lv, int t, LdsInts tab, const bool (&act)[NC],
                                   int (&cells)[NC], int (&res)[NC])
{
    if constexpr (NC == 2) {
        // two candidates per lane: the packed 16-bit DP (register strings only)
        if (yrows) vsp_seg2<MAXW, true, TS>(U, lu, V, lv, t, tab, act, cells, res);
        else vsp_seg2<MAXW, false, TS>(U, lu, V, lv, t, tab, act, cells, res);
    } else {
        if (yrows) vsp_seg<MAXW, true, NC, TS>(U, lu, V, lv, t, tab, act, cells, res);
        else vsp_seg<MAXW, false, NC, TS>(U, lu, V, lv, t, tab, act, cells, res);
    }
}

// band width t + 1 for a uniform t <= 8 below the width class, else the class width GMAXW
template <int GMAXW, int NC, int TS, typename LaneChars>
__device__ inline void vsp_seg_dispatch(bool yrows, LdsChars U, int lu, const LaneChars (&V)[NC],
                                        int lv, int t, LdsInts tab, const bool (&act)[NC],
                                        int (&cells)[NC], int (&res)[NC])
{
    if (t + 1 >= GMAXW || t > 8) {
        vsp_seg_any<GMAXW, NC, TS>(yrows, U, lu, V, lv, t, tab, act, cells, res);
        return;
    }
#define PJ_SEG_CASE(T)                                                                      \
    case T:                                                                                 \
        if constexpr (T + 1 < GMAXW)                                                        \
            vsp_seg_any<T + 1, NC, TS>(yrows, U, lu, V, lv, t, tab, act, cells, res);       \
        break;
    switch (t) {
    PJ_SEG_CASE(0)
    PJ_SEG_CASE(1)
    PJ_SEG_CASE(2)
    PJ_SEG_CASE(3)
    PJ_SEG_CASE(4)
    PJ_SEG_CASE(5)
    PJ_SEG_CASE(6)
    PJ_SEG_CASE(7)
    PJ_SEG_CASE(8)
    default: break;
    }
#undef PJ_SEG_CASE
}

template <int MAXW, int KF, int TS>
__device__ inline void vsp_lane_or(bool yrows, LdsChars U, int lu, LdsLaneChars V, int lv, int t,
                                   LdsInts tab, bool act, int& cells, int& res)
{
    if (yrows) vsp_lane<MAXW, KF, true, TS>(U, lu, V, lv, t, tab, act, cells, res);
    else vsp_lane<MAXW, KF, false, TS>(U, lu, V, lv, t, tab, act, cells, res);
}

// vsp_lane at width t + 1 (the width class GMAXW when t + 1 reaches it); for t <= 4 the band
// index of the final cell, (t + |lu - lv|) / 2, is a compile-time constant too
template <int GMAXW, int TS>
__device__ inline void vsp_lane_dispatch(bool yrows, LdsChars U, int lu, LdsLaneChars V, int lv,
                                         int t, LdsInts tab, bool act, int& cells, int& res)
{
    static_assert(GMAXW >= 5 && GMAXW <= 9, "narrow width classes only");
    const int delta = lu > lv ? lu - lv : lv - lu;
    if (delta > t) {
        cells = 0;
        res = t + 1;
        return;
    }
    const int kf = (t + delta) >> 1;
    cells = 0;                                   // t < GMAXW always; kept defined regardless
    res = t + 1;
#define PJ_LANE(W, K) vsp_lane_or<W, K, TS>(yrows, U, lu, V, lv, t, tab, act, cells, res)
    switch (t) {
    case 0: PJ_LANE(1, 0); return;
    case 1: if (kf == 0) PJ_LANE(2, 0); else PJ_LANE(2, 1); return;
    case 2: if (kf == 1) PJ_LANE(3, 1); else PJ_LANE(3, 2); return;
    case 3: if (kf == 1) PJ_LANE(4, 1); else if (kf == 2) PJ_LANE(4, 2); else PJ_LANE(4, 3); return;
    case 4: if (kf == 2) PJ_LANE(5, 2); else if (kf == 3) PJ_LANE(5, 3); else PJ_LANE(5, 4); return;
    default: break;
    }
    if constexpr (GMAXW > 5) {
        if (t == 5 && GMAXW > 6) { PJ_LANE(6 < GMAXW ? 6 : GMAXW, -1); return; }
        if (t == 6 && GMAXW > 7) { PJ_LANE(7 < GMAXW ? 7 : GMAXW, -1); return; }
        if (t == 7 && GMAXW > 8) { PJ_LANE(8 < GMAXW ? 8 : GMAXW, -1); return; }
        PJ_LANE(GMAXW, -1);
    }
#undef PJ_LANE
}

template <int GMAXW, int REGY, int NCT>
__global__ __launch_bounds__(kBlock) void k_verify_segs(VerifyParams V, Div div,
                                                        const Hit* __restrict__ big,
                                                        const uint32_t* __restrict__ segp,
                                                        uint64_t /* hits (unused) */,
                                                        uint64_t nseg,
                                                        const uint32_t* __restrict__ first,
                                                        uint64_t nchunks, uint32_t seg_chunk,
                                                        unsigned long long* ticket)
{
    // NC candidates per lane: a list segment has 64 * NC members
    constexpr int NC = (REGY > 0 && GMAXW <= 9) ? NCT : 1;
    constexpr uint32_t SEG = 64u * NC;
    // one candidate per lane and indexed strings of at most REGY bytes: each lane copies its
    // string into an LDS slot of its own, from which the band DP reads it (vsp_lane)
    constexpr bool LANE = REGY > 0 && NC == 1 && GMAXW <= 9;
    // slot stride REGY + 4 bytes, an odd number of words, so a wave's reads at one offset hit
    // distinct banks; 16 bytes before the first slot and after the last absorb the reads of
    // columns outside the string (at most 4 bytes before a string, at most 12 after it: a DP
    // block reads up to 2 * MAXW - 2 - kfin past the part, with kfin >= t / 2)
    constexpr int SL = REGY + 4, YPAD = 16, YTAIL = 16;
    constexpr int kCap = 96;                               // pairs buffered per wave
    __shared__ uint64_t s_acc[kWaves][kCap];
    // the current probe string; the band DP reads at most 2 * MAXW bytes past a part's end
    // (vsp_seg and vsp_lane up to width 9; the wider classes keep 128).  An indexed string of
    // at most REGY bytes has probes of at most REGY + tau bytes.
    constexpr int XMAX = REGY > 0 ? REGY + (GMAXW <= 9 ? GMAXW - 1 : kTauMax) : kLenMax;
    constexpr int XPAD = GMAXW <= 9 ? 32 : 128;
    __shared__ uint32_t s_x[kWaves][(XMAX + 1 + XPAD + 3) / 4];
    __shared__ uint32_t s_q[kWaves][2 * SEG];             // left-part survivors
    // band tables of the current hit's two parts (row 0, distance offsets, first window, and
    // the rows of vsp_lane)
    constexpr int BTS = (GMAXW + 3) & ~3;
    constexpr int CT = LANE ? REGY + 4 : 0;               // cells table: rows 0 .. nr <= REGY
    __shared__ __attribute__((aligned(16))) int s_band[kWaves][2][6 * BTS + CT];
    constexpr int YW = LANE ? (YPAD + 64 * SL + YTAIL) / 4 : 1;
    __shared__ __attribute__((aligned(16))) uint32_t s_y[kWaves][YW];   // lane slots (LANE)
    WaveAppender<uint64_t, kCap> acc{s_acc[threadIdx.x >> 6], 0};
    const int lane = threadIdx.x & 63;
    uint32_t* sx = s_x[threadIdx.x >> 6];
    uint32_t* sq = s_q[threadIdx.x >> 6];
    const __attribute__((address_space(3))) uint8_t* xl8 =
        (const __attribute__((address_space(3))) uint8_t*)(sx);
    // this lane's slot (LANE)
    __attribute__((address_space(3))) uint32_t* ysw =
        (__attribute__((address_space(3))) uint32_t*)(s_y[threadIdx.x >> 6]) +
        (YPAD + lane * SL) / 4;
    const __attribute__((address_space(3))) uint8_t* ys8 =
        (const __attribute__((address_space(3))) uint8_t*)(ysw);
    // wave id as a scalar, so that everything derived from it is known to be wave-uniform
    const uint64_t wave = (uint64_t)blockIdx.x * kWaves +
                          (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t nwaves = (uint64_t)gridDim.x * kWaves;
    uint64_t my_cells = 0, my_miss = 0;
    // a wave's first chunk is its own, the others are taken as waves come free: lists differ in
    // work far more than chunks do in number
    uint32_t tried = 0;
    uint64_t ch = wave;
    while (ch < nchunks) {
        uint64_t sg_i = ch * seg_chunk;
        const uint64_t sg_end = (sg_i + seg_chunk < nseg) ? sg_i + seg_chunk : nseg;
        uint32_t h = uniform_load(first + ch);
        uint32_t sidx = (uint32_t)(sg_i - uniform_load(segp + h));
        while (sg_i < sg_end) {
            // everything about the hit is wave-uniform: probe string, slot, both parts
            const uint32_t* hw = reinterpret_cast<const uint32_t*>(big + h);
            const uint32_t gx = uniform_load(hw), start = uniform_load(hw + 1);
            const uint32_t count = uniform_load(hw + 2), meta = uniform_load(hw + 3);
            int tau = V.tau;
            const uint32_t* vals = V.vals;
            Div dv = div;
            if (V.q_tau) {
                tau = uniform_load(V.q_tau + gx);
                const IndexRef* rf = V.refs + tau;
                vals = uniform_load(&rf->vals);
                dv.d = (uint32_t)(tau + 1);
                dv.m = uniform_load(&rf->div_m);
            }
            const int p = (int)(meta & 2047u) + 1;
            const int i = (int)((meta >> 11) & 63u) + 1;
            const int l = (int)(meta >> 17);
            const int n = __builtin_amdgcn_readfirstlane((int)V.x_slen[gx]);
            const uint8_t* x = V.x_arena + uniform_load(V.x_gbase + n) +
                               (int64_t)(gx - (uint32_t)uniform_load(V.x_lenstart + n)) * stride_of(n);
            const int64_t ybase = uniform_load(V.y_gbase + l) -
                                  (int64_t)uniform_load(V.y_lenstart + l) * stride_of(l);
            const Seg sgm = partition_seg(l, i, tau, dv);
            // stage x in the wave's LDS buffer (its slot is 16-byte aligned); the previous
            // hit's reads were issued before these writes, and LDS requests of a wave complete
            // in order
            {
                const uint32_t* xw = reinterpret_cast<const uint32_t*>(x);
                for (int q = lane; q < ((n + 3) >> 2); q += 64) sx[q] = xw[q];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            // left parts: x[1, p-1] vs y[1, p_i-1] with t = i-1; right parts after the segment
            // with t = tau+1-i (Algorithm 3)
            const int tl = i - 1, tr = tau + 1 - i;
            const int ry = sgm.p - 1 + sgm.len, rx = p - 1 + sgm.len;
            // the previous hit's table reads were issued before these writes
            __attribute__((address_space(3))) int* tab_l =
                (__attribute__((address_space(3))) int*)s_band[threadIdx.x >> 6][0];
            __attribute__((address_space(3))) int* tab_r =
                (__attribute__((address_space(3))) int*)s_band[threadIdx.x >> 6][1];
            band_table(LdsChars{xl8}, p - 1, sgm.p - 1, tl, lane, BTS, NC == 2, tab_l, CT);
            band_table(LdsChars{xl8 + rx}, n - rx, l - ry, tr, lane, BTS, NC == 2, tab_r, CT);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const uint32_t hsegs = (count + SEG - 1) / SEG;
            const uint64_t left_in_chunk = sg_end - sg_i;
            const uint32_t s_stop = (uint64_t)(hsegs - sidx) < left_in_chunk
                                        ? hsegs : sidx + (uint32_t)left_in_chunk;
            // REGY > 0: the whole indexed string (at most REGY bytes, 16-byte aligned slot) goes
            // to registers with wide loads and is read at wave-uniform offsets
            // With the index's inline copies a list's strings are contiguous (entry e at
            // yinl + e * stride), so a segment's loads are coalesced and need no list entry first
            const uint8_t* yinl = nullptr;
            if (REGY > 0 && V.y_inl) yinl = V.y_inl + uniform_load(V.y_inl_base + l);
            // REGY > 0: the indexed string's words (at most REGY bytes) go to registers, or,
            // with LANE, straight into the lane's LDS slot (a wave's LDS requests complete in
            // order: the DP's reads see these words, the previous DP's reads did not); words
            // past the string are not loaded
            auto load_y = [&](uint32_t g, uint32_t e, uint32_t* yr) -> const uint8_t* {
                const uint8_t* y = yinl ? yinl + (int64_t)e * stride_of(l)
                                        : V.y_arena + ybase + (int64_t)g * stride_of(l);
                if constexpr (LANE) {
                    // every load first, then the writes: one wait for all of them.  A class
                    // of REGY = 40 loads 48 bytes (inside the 48-byte stride of its strings)
                    // and writes the slot's 10 words only
                    constexpr int NQ = (REGY + 15) / 16;
                    const uint4* yq = reinterpret_cast<const uint4*>(y);
                    uint4 v[NQ];
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
                        if (q * 16 < l) v[q] = yq[q];
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        if (q * 16 < l) {
                            ysw[4 * q] = v[q].x;
                            if (16 * q + 4 < REGY) ysw[4 * q + 1] = v[q].y;
                            if (16 * q + 8 < REGY) ysw[4 * q + 2] = v[q].z;
                            if (16 * q + 12 < REGY) ysw[4 * q + 3] = v[q].w;
                        }
                    }
                } else if (REGY > 0) {
                    const uint4* yq = reinterpret_cast<const uint4*>(y);
#pragma unroll
                    for (int q = 0; q < (REGY > 0 ? REGY / 16 : 0); ++q) {
                        const uint4 v = (q * 16 < l) ? yq[q] : make_uint4(0u, 0u, 0u, 0u);
                        yr[4 * q] = v.x; yr[4 * q + 1] = v.y;
                        yr[4 * q + 2] = v.z; yr[4 * q + 3] = v.w;
                    }
                }
                return y;
            };
            // Two phases per hit: the left parts of each segment, then the right parts of the
            // survivors, taken SEG at a time from a wave-private queue, so that a wave's
            // right-part rows are not spent on lanes whose left part already failed.  Each
            // iteration runs one band DP: a left step (next segment) or a right batch (SEG queued
            // survivors, or the rest once the segments are done).
            // A part whose two strings are both empty passes with no cells (ED 0 <= t): the
            // left parts of slot 1 (p = p_1 = 1) and the right parts of slot tau+1 (x and y both
            // end with the segment).  Then the other part runs directly on the segment members,
            // without the queue.
            const bool left_trivial = (p == 1) && (sgm.p == 1);
            const bool right_trivial = (rx == n) && (ry == l);
            uint32_t qn = 0;    // queued survivors (wave-uniform)
            for (;;) {
                const bool right = left_trivial ? sidx < s_stop
                                                : (qn >= SEG || (sidx >= s_stop && qn > 0));
                if (!right && sidx >= s_stop) break;
                const bool from_queue = right && !left_trivial;
                const uint32_t k = from_queue ? (qn < SEG ? qn : SEG) : 0;
                if (from_queue) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
                uint32_t gy[NC], ent[NC];
                uint32_t yr[NC][(REGY > 0 && !LANE) ? REGY / 4 : 1];
                const uint8_t* y[NC];
                bool ok[NC];
                bool anyok = false;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const uint32_t slot = (uint32_t)c * 64u + (uint32_t)lane;
                    const uint32_t member = sidx * SEG + slot;
                    ok[c] = from_queue ? slot < k : member < count;
                    // every lane takes a valid candidate (an inactive one repeats the first
                    // queued candidate, k >= 1, or the hit's last member, count >= 1), so the
                    // loads below need no per-lane branch; only active lanes count.  The queue
                    // holds index entries (inline copies) or string positions.
                    uint32_t src;
                    if (from_queue) src = sq[ok[c] ? slot : 0u];     // slot < 2 * SEG
                    else src = start + (ok[c] ? member : count - 1u);
                    if (yinl) {
                        ent[c] = src;
                        // string positions are needed only to emit pairs
                        gy[c] = (right || right_trivial) ? vals[src] : 0u;
                    } else {
                        ent[c] = 0;
                        gy[c] = from_queue ? src : vals[src];
                    }
                    y[c] = load_y(gy[c], ent[c], yr[c]);
                    if (!from_queue && sgm.len > V.exact_len) {
                        // hashed key: compare the segment bytes before extension
                        // verification, which skips the segment
                        const LdsChars xs{xl8 + (p - 1)};
                        bool same = true;
                        if constexpr (LANE) {
                            const LdsLaneChars yc{ys8 + (sgm.p - 1)};
                            for (int q = 0; q < sgm.len; ++q) same &= (xs[q] == yc[q]);
                        } else if constexpr (REGY > 0) {
                            const RegChars yc{yr[c], sgm.p - 1};
                            for (int q = 0; q < sgm.len; ++q) same &= (xs[q] == yc[q]);
                        } else {
                            for (int q = 0; q < sgm.len; ++q)
                                same &= (xs[q] == (int)y[c][sgm.p - 1 + q]);
                        }
                        my_miss += (ok[c] && !same) ? 1 : 0;
                        ok[c] = ok[c] && same;
                    }
                    anyok = anyok || ok[c];
                }
                if (anyok) {
                    const int xo = right ? rx : 0, xl = right ? n - rx : p - 1;
                    const int yo = right ? ry : 0, yl = right ? l - ry : sgm.p - 1;
                    const int tt = right ? tr : tl;
                    int cl[NC], d[NC];
                    if constexpr (LANE) {
                        vsp_lane_dispatch<GMAXW, BTS>(yl <= xl, LdsChars{xl8 + xo}, xl,
                                                      LdsLaneChars{ys8 + yo}, yl, tt,
                                                      right ? tab_r : tab_l, ok[0], cl[0], d[0]);
                    } else if constexpr (REGY > 0) {
                        RegChars vc[NC];
#pragma unroll
                        for (int c = 0; c < NC; ++c) vc[c] = RegChars{yr[c], yo};
                        vsp_seg_dispatch<GMAXW, NC, BTS>(yl <= xl, LdsChars{xl8 + xo}, xl, vc,
                                                         yl, tt, right ? tab_r : tab_l, ok, cl,
                                                         d);
                    } else {
                        GlobalChars vc[NC];
#pragma unroll
                        for (int c = 0; c < NC; ++c) vc[c] = GlobalChars{y[c] + yo};
                        vsp_seg_dispatch<GMAXW, NC, BTS>(yl <= xl, LdsChars{xl8 + xo}, xl, vc,
                                                         yl, tt, right ? tab_r : tab_l, ok, cl,
                                                         d);
                    }
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        my_cells += (uint64_t)cl[c];
                        ok[c] = ok[c] && d[c] <= tt;
                    }
                }
                if (right || right_trivial) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        acc.push(ok[c], ((uint64_t)gx << 32) | gy[c], V.out, V.out_cap,
                                 &V.counters[3]);
                }
                if (!from_queue) {
                    ++sidx;
                    ++sg_i;
                }
                if (from_queue) {
                    // move the rest of the queue (entries SEG .. qn-1) to its front, all reads
                    // before the writes; every lane moves a word, those past the rest are free
                    const uint32_t rest = qn - k;
                    uint32_t mv[NC];
#pragma unroll
                    for (int c = 0; c < NC; ++c) mv[c] = sq[SEG + (uint32_t)(c * 64 + lane)];
#pragma unroll
                    for (int c = 0; c < NC; ++c) sq[(uint32_t)(c * 64 + lane)] = mv[c];
                    qn = rest;
                } else if (!right && !right_trivial) {
                    // survivors appended in lane order; a left step starts with qn < SEG, so
                    // the last word, 2 * SEG - 1, is never an entry and takes the other lanes'
                    // writes
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const uint64_t surv = __builtin_amdgcn_ballot_w64(ok[c]);
                        const uint32_t at = qn + __builtin_amdgcn_mbcnt_hi(
                                                     (uint32_t)(surv >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)surv, 0u));
                        sq[ok[c] ? at : 2u * SEG - 1u] = yinl ? ent[c] : gy[c];
                        qn += (uint32_t)__builtin_popcountll(surv);
                    }
                }
            }
            ++h;
            sidx = 0;
        }
        ch = next_chunk(ticket, tried, nwaves, nchunks);
    }
    block_flush(acc, V.out, V.out_cap, &V.counters[3]);
    unsigned long long* line = stat_line(V.counters, V.shards);
    block_add(&line[7], my_cells);
    block_add(&line[5], my_miss);
}

// ------------------------------------------------------------------------------------------
// Short strings (length <= tau): not partitionable (footnote to Sec. 3.1).  One block per short
// string y of the indexed set; its partners are the probe-set strings in the length window
// [|y| - tau, |y| + tau] -- a contiguous range of sorted positions.  In a self-join a pair of
// two short strings is taken once (from the later one).
// ------------------------------------------------------------------------------------------

// ------------------------------------------------------------------------------------------
// Shared-prefix verification (Sec. 5.3).  The paper walks an inverted list in alphabetical
// order and lets each member's DP start from the rows its left (right) part shares with the
// previous member's.  In a wave the 64 lanes advance row by row together, so sharing rows
// between lanes saves nothing; here a lane walks a chain of kChainMembers consecutive members
// of a content-ordered list on its own, as the paper's loop does, keeping its previous
// member's first kShareRows rows per side in LDS.  Lanes of a wave take consecutive chains
// (the same list, or the next big lists).
// ------------------------------------------------------------------------------------------

// chains of one big hit: the whole list is walked in content order, so for a self-join's list
// of the probe string's own length the members visited after it are skipped one by one
__global__ __launch_bounds__(kBlock) void k_chain_counts(const Hit* __restrict__ big, uint64_t nbig,
                                                         const uint16_t* __restrict__ x_slen,
                                                         const uint32_t* __restrict__ runlen,
                                                         int self, uint32_t* __restrict__ chains)
{
    const uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= nbig) return;
    const Hit h = big[k];
    const int l = (int)(h.meta >> 17);
    const uint32_t full = (self && l == (int)x_slen[h.gx]) ? runlen[h.start] : h.count;
    chains[k] = (full + kChainMembers - 1u) / kChainMembers;
}

template <int MAXW>
__global__ __launch_bounds__(kBlock) void k_verify_chains(VerifyParams V, Div div,
                                                          const Hit* __restrict__ big,
                                                          const unsigned long long* __restrict__ cprefix,
                                                          uint64_t nbig, uint64_t nchains,
                                                          const uint32_t* __restrict__ first,
                                                          uint64_t nchunks)
{
    constexpr int NW = (MAXW + 7) / 8;
    __shared__ uint64_t s_acc[kWaves][kAppendCap];
    __shared__ uint32_t s_mat[kWaves][2][kShareRows * NW * 64];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    WaveAppender<uint64_t, kAppendCap> acc{s_acc[wv], 0};
    __attribute__((address_space(3))) uint32_t* matL =
        (__attribute__((address_space(3))) uint32_t*)(s_mat[wv][0]) + lane;
    __attribute__((address_space(3))) uint32_t* matR =
        (__attribute__((address_space(3))) uint32_t*)(s_mat[wv][1]) + lane;
    const uint64_t wave = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const uint64_t nwaves = ((uint64_t)gridDim.x * kBlock) >> 6;
    uint64_t my_cells = 0, my_miss = 0, my_srows = 0, my_scells = 0;
    const uint64_t le_mask = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    for (uint64_t ch = wave; ch < nchunks; ch += nwaves) {
        const uint64_t c0 = ch * 64ull;
        const uint64_t h = first[ch];
        // the chain of each lane: boundaries of hits h .. h + 63 inside [c0, c0 + 64)
        const uint64_t hk = h + (uint64_t)lane;
        const unsigned long long bk = (hk < nbig) ? cprefix[hk + 1] : ~0ull;
        const uint64_t rel = bk - c0;
        const uint64_t M = wave_or64(rel < 64 ? (1ull << rel) : 0ull);
        const int off = __popcll(M & le_mask);
        const unsigned long long bprev = __shfl(bk, off > 0 ? off - 1 : 0, 64);
        const unsigned long long hs = (off == 0) ? cprefix[h] : bprev;
        const uint64_t c = c0 + (uint64_t)lane;
        const bool valid = c < nchains;
        Hit hit{0, 0, 0, 0};
        int n = 0, l = 0, p = 1, i = 1;
        uint32_t m0 = 0, m1 = 0;
        const uint8_t* x = nullptr;
        Seg sg{1, 0};
        if (valid) {
            hit = big[h + (uint64_t)off];
            p = (int)(hit.meta & 2047u) + 1;
            i = (int)((hit.meta >> 11) & 63u) + 1;
            l = (int)(hit.meta >> 17);
            n = V.x_slen[hit.gx];
            x = V.x_arena + V.x_gbase[n] + (int64_t)(hit.gx - V.x_lenstart[n]) * stride_of(n);
            const uint32_t full = (V.self && l == n) ? V.runlen[hit.start] : hit.count;
            m0 = (uint32_t)(c - hs) * (uint32_t)kChainMembers;
            m1 = min(m0 + (uint32_t)kChainMembers, full);
            sg = partition_seg(l, i, V.tau, div);
        }
        const int tl = i - 1, tr = V.tau + 1 - i;
        const int ry = sg.p - 1 + sg.len, rx = p - 1 + sg.len;
        SharePrev pl{nullptr, 0, 0, 0, 0}, pr{nullptr, 0, 0, 0, 0};
        for (int it = 0; it < kChainMembers; ++it) {
            const uint32_t m = m0 + (uint32_t)it;
            bool cand = valid && m < m1;
            uint32_t gy = 0;
            if (cand) {
                gy = V.svals[hit.start + m];
                if (V.self && l == n && gy >= hit.gx) cand = false;    // visited after x
            }
            bool pass = false;
            if (cand) {
                const uint8_t* y = V.y_arena + V.y_gbase[l] +
                                   (int64_t)(gy - V.y_lenstart[l]) * stride_of(l);
                bool same = true;
                if (sg.len > V.exact_len)
                    for (int k = 0; k < sg.len; ++k) same &= (x[p - 1 + k] == y[sg.p - 1 + k]);
                if (!same) {
                    my_miss += 1;
                } else {
                    const int dl = share_part<MAXW>(y, sg.p - 1, x, p - 1, tl, pl, matL, my_cells,
                                                    my_srows, my_scells);
                    if (dl <= tl) {
                        const int dr = share_part<MAXW>(y + ry, l - ry, x + rx, n - rx, tr, pr,
                                                        matR, my_cells, my_srows, my_scells);
                        pass = dr <= tr;
                    }
                }
            }
            acc.push(pass, ((uint64_t)hit.gx << 32) | gy, V.out, V.out_cap, &V.counters[3]);
        }
    }
    block_flush(acc, V.out, V.out_cap, &V.counters[3]);
    unsigned long long* line = stat_line(V.counters, V.shards);
    block_add(&line[4], my_cells);
    block_add(&line[5], my_miss);
    block_add(&line[8], my_srows);
    block_add(&line[9], my_scells);
}

// Content order of the index entries: the first 8 bytes of each entry's string, big-endian,
// so that comparing keys compares the strings' first 8 bytes; idx = entry number.
__global__ __launch_bounds__(kBlock) void k_prefix8_keys(const uint32_t* __restrict__ vals, int64_t E,
                                                         const uint8_t* __restrict__ sarena,
                                                         const uint16_t* __restrict__ slen,
                                                         const int32_t* __restrict__ lenstart,
                                                         const int64_t* __restrict__ gbase,
                                                         uint64_t* __restrict__ keys,
                                                         uint32_t* __restrict__ idx)
{
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= E) return;
    const uint32_t g = vals[e];
    const int l = slen[g];
    const uint8_t* w = sarena + gbase[l] + (int64_t)(g - lenstart[l]) * stride_of(l);
    uint64_t k = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) k = (k << 8) | (uint64_t)(b < l ? w[b] : 0);
    keys[e] = k;
    idx[e] = (uint32_t)e;
}

__global__ __launch_bounds__(kBlock) void k_gather_keys(const uint64_t* __restrict__ keys,
                                                        const uint32_t* __restrict__ idx, int64_t E,
                                                        uint64_t* __restrict__ out)
{
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e < E) out[e] = keys[idx[e]];
}

__global__ __launch_bounds__(kBlock) void k_gather_vals(const uint32_t* __restrict__ vals,
                                                        const uint32_t* __restrict__ idx, int64_t E,
                                                        uint32_t* __restrict__ out)
{
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e < E) out[e] = vals[idx[e]];
}

__global__ __launch_bounds__(kBlock) void k_run_lengths(const uint32_t* __restrict__ runstart,
                                                        uint32_t nruns, uint32_t E,
                                                        uint32_t* __restrict__ runlen)
{
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= nruns) return;
    const uint32_t st = runstart[r];
    runlen[st] = ((r + 1 < nruns) ? runstart[r + 1] : E) - st;
}

// ------------------------------------------------------------------------------------------
// Long-string verification.  A candidate's part DP runs for hundreds of rows when it passes and
// stops after a few when it does not, so 64 candidates in lockstep leave most lanes idle.  Here the
// candidates of the small lists are materialised in slot order (one (tau_l, tau_r) per slot, so a
// wave's 64 tasks share the band width class).  Their left parts' first rows run a candidate a lane
// (k_verify_first), which ends most; the others, and the right parts, are taken a diagonal a lane
// (k_verify_far), which costs by differences and not by rows.
// ------------------------------------------------------------------------------------------

constexpr int kContMaxRows = 64;     // rows staged at a time
constexpr int kContW = 33;           // widest band class
// 16-byte blocks staged per lane: A needs kContMaxRows + 15 bytes, B kContW + kContMaxRows + 15 + 15
constexpr int kStageA = (kContMaxRows + 15 + 15) / 16;
constexpr int kStageB = (kContW + kContMaxRows + 15 + 15) / 16;

// A task: {gx, gy, meta, n} and the byte offsets of x and y in their arenas.
struct LongRec {
    uint4 a;        // gx, gy, meta (p, i, l), n = |x|
    uint4 b;        // x offset (lo, hi), y offset (lo, hi)
};
// per slot (i - 1): number of candidates of the small-list hits
__global__ __launch_bounds__(kBlock) void k_long_slot_counts(const Hit* __restrict__ hits, uint64_t nh,
                                                             uint32_t* __restrict__ slot_cnt)
{
    __shared__ uint32_t s_cnt[64];
    if (threadIdx.x < 64) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    for (uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x; k < nh;
         k += (uint64_t)gridDim.x * kBlock)
        atomicAdd(&s_cnt[(hits[k].meta >> 11) & 63u], hits[k].count);
    __syncthreads();
    if (threadIdx.x < 64 && s_cnt[threadIdx.x]) atomicAdd(&slot_cnt[threadIdx.x], s_cnt[threadIdx.x]);
}

// one wave: exclusive scan of the 64 slot counts into off[0..64], cursor = off
__global__ void k_long_slot_offsets(const uint32_t* __restrict__ slot_cnt, uint32_t* __restrict__ off,
                                    uint32_t* __restrict__ cursor)
{
    const int lane = threadIdx.x;
    const uint32_t c = slot_cnt[lane];
    const uint32_t incl = wave_incl_scan(c);
    off[lane] = incl - c;
    cursor[lane] = incl - c;
    if (lane == 63) off[64] = incl;
}

// Candidates of the small-list hits to their slots' regions.  A block walks a contiguous range
// of hits twice: first counting its candidates per slot in LDS, then, after reserving each
// slot's share with one global atomic, writing them (a global atomic per hit on the 64 slot
// cursors would serialise).
__global__ __launch_bounds__(kBlock) void k_long_scatter(const Hit* __restrict__ hits, uint64_t nh,
                                                         const uint32_t* __restrict__ vals,
                                                         const uint16_t* __restrict__ x_slen,
                                                         const int32_t* __restrict__ x_lenstart,
                                                         const int64_t* __restrict__ x_gbase,
                                                         const int32_t* __restrict__ y_lenstart,
                                                         const int64_t* __restrict__ y_gbase,
                                                         uint32_t* __restrict__ cursor,
                                                         LongRec* __restrict__ cands)
{
    __shared__ uint32_t s_cnt[64];
    __shared__ uint32_t s_pos[64];
    const uint64_t per = (nh + gridDim.x - 1) / gridDim.x;
    const uint64_t h0 = (uint64_t)blockIdx.x * per;
    const uint64_t h1 = min(h0 + per, nh);
    if (threadIdx.x < 64) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    for (uint64_t k = h0 + threadIdx.x; k < h1; k += kBlock) {
        const Hit h = hits[k];
        atomicAdd(&s_cnt[(h.meta >> 11) & 63u], h.count);
    }
    __syncthreads();
    if (threadIdx.x < 64)
        s_pos[threadIdx.x] = s_cnt[threadIdx.x] ? atomicAdd(&cursor[threadIdx.x], s_cnt[threadIdx.x]) : 0u;
    __syncthreads();
    for (uint64_t k = h0 + threadIdx.x; k < h1; k += kBlock) {
        const Hit h = hits[k];
        const int n = x_slen[h.gx];
        const int l = (int)(h.meta >> 17);
        const uint64_t xo = (uint64_t)(x_gbase[n] + (int64_t)(h.gx - x_lenstart[n]) * stride_of(n));
        const uint32_t base = atomicAdd(&s_pos[(h.meta >> 11) & 63u], h.count);
        for (uint32_t m = 0; m < h.count; ++m) {
            const uint32_t gy = vals[h.start + m];
            const uint64_t yo = (uint64_t)(y_gbase[l] + (int64_t)(gy - y_lenstart[l]) * stride_of(l));
            LongRec r;
            r.a = make_uint4(h.gx, gy, h.meta, (uint32_t)n);
            r.b = make_uint4((uint32_t)xo, (uint32_t)(xo >> 32), (uint32_t)yo, (uint32_t)(yo >> 32));
            cands[base + m] = r;
        }
    }
}

// Chunks of the slots' tasks: counts by slot (lane = slot), `per` tasks a chunk (by slot too); finds a
// chunk's slot and its range in the slot's region.
struct SlotChunks {
    uint32_t count, per, chunks, incl, total;
    __device__ SlotChunks(const uint32_t* counts, int slots, uint32_t per_) : per(per_)
    {
        const int lane = threadIdx.x & 63;
        count = lane < slots ? counts[lane] : 0u;
        chunks = (count + per - 1) / per;
        incl = wave_incl_scan(chunks);
        total = __shfl(incl, 63, 64);
    }
    __device__ int find(uint32_t ch, uint32_t* b0, uint32_t* b1) const
    {
        const int slot = __popcll(__ballot(incl <= ch));
        const uint32_t p = __shfl(per, slot, 64);
        *b0 = (ch - __shfl(incl - chunks, slot, 64)) * p;
        *b1 = min(*b0 + p, (uint32_t)__shfl(count, slot, 64));
        return slot;
    }
};

// rec of the flagged lanes to the slot's region of out
__device__ inline void append_tasks(bool flag, const LongRec& rec, LongRec* __restrict__ out,
                                    uint32_t* count)
{
    const uint64_t m = __ballot(flag);
    if (!m) return;
    uint32_t base = 0;
    if ((threadIdx.x & 63) == 0) base = atomicAdd(count, (uint32_t)__popcll(m));
    base = __shfl(base, 0, 64);
    if (flag) out[base + (uint32_t)__popcll(m & lanemask_lt())] = rec;
}

// The candidates [b0, b1) of one slot for one wave (one per lane): up to K rows of each one's left
// part DP on M values in diagonal coordinates (band index k holds column j = i - a + k of row i;
// up = index k + 1, left = k - 1 of this row, diagonal = k; cells outside the band or left of
// column 0 start large and only see large inputs, so column 0 follows from the recurrence;
// indices right of column nc never feed a cell inside the matrix).  The expected distance of
// index k is M + |b - k| (b = a + Delta, the final cell's index); a row whose smallest one
// exceeds t stops the DP (Lemma 4).  The characters come from the lane's LDS stage (element q at
// stage[q * 64]): A[row + q] for q < kContMaxRows, then B[row - a + q] (256 outside B).  Parts that
// pass go to rout, parts that are not done to cout (whole, k_verify_far starts them anew).
template <int MAXW>
__device__ inline void first_rows(const VerifyParams& V, const Div& div, int slot,
                                  const LongRec* __restrict__ fin, uint32_t b0, uint32_t b1, int K,
                                  LongRec* __restrict__ cout, uint32_t* __restrict__ cout_cnt,
                                  LongRec* __restrict__ rout, uint32_t* __restrict__ rout_cnt,
                                  uint32_t qbase,
                                  __attribute__((address_space(3))) uint32_t* stage32,
                                  uint64_t& my_cells, uint64_t& my_miss)
{
    constexpr int BIG = 1 << 20;
    const int lane = threadIdx.x & 63;
    // the lane's 16-byte blocks: block q at byte (q * 64 + lane) * 16 of the wave's stage
    const __attribute__((address_space(3))) uint8_t* stage8 =
        (const __attribute__((address_space(3))) uint8_t*)stage32;
    const int i = slot + 1;
    const int t = i - 1;
    const uint32_t k = b0 + (uint32_t)lane;
    bool act = k < b1;
    LongRec rec;
    rec.a = make_uint4(0u, 0u, 0u, 0u);
    rec.b = rec.a;
    int M[MAXW];                                          // every lane runs the row loop
#pragma unroll
    for (int q = 0; q < MAXW; ++q) M[q] = BIG;
    int row = 0, nr = 0, nc = 0, a = 0, b = 0, st = 0;    // st: 0 running, 1 pass, 2 fail, 3 none
    const uint8_t* A = nullptr;
    const uint8_t* B = nullptr;
    const uint8_t* A_end = nullptr;     // end of the padded slot of A's / B's string
    const uint8_t* B_end = nullptr;
    if (act) {
        rec = fin[k];
        const uint32_t meta = rec.a.z;
        const int p = (int)(meta & 2047u) + 1;
        const int l = (int)(meta >> 17);
        const int n = (int)rec.a.w;
        const uint8_t* x = V.x_arena + ((uint64_t)rec.b.y << 32 | rec.b.x);
        const uint8_t* y = V.y_arena + ((uint64_t)rec.b.w << 32 | rec.b.z);
        const Seg sg = partition_seg(l, i, V.tau, div);
        const int lr = sg.p - 1, ls = p - 1;
        const uint8_t* yend = y + stride_of(l);
        const uint8_t* xend = x + stride_of(n);
        if (lr <= ls) { A = y; nr = lr; B = x; nc = ls; A_end = yend; B_end = xend; }
        else          { A = x; nr = ls; B = y; nc = lr; A_end = xend; B_end = yend; }
        const int delta = nc - nr;
        a = (t - delta) >> 1;
        b = (t + delta) >> 1;
        bool ok = true;
        if (sg.len > V.exact_len) {
            for (int q = 0; q < sg.len; ++q) ok &= (x[p - 1 + q] == y[sg.p - 1 + q]);
            if (!ok) my_miss += 1;
        }
        if (!ok) st = 3;                                   // not a candidate
        else if (delta > t) st = 2;                        // no row
        else if (nr == 0) st = (nc <= t) ? 1 : 2;
#pragma unroll
        for (int q = 0; q < MAXW; ++q) {
            const int j = q - a;
            M[q] = (j >= 0 && j <= min(nc, b)) ? j : BIG;
        }
    }
    // the rows in sub-blocks of kContMaxRows: each stages its characters (the 16-byte
    // blocks holding A[row .. row + 64) and B[max(row - a, 0) .. row - a + MAXW + 64), each block
    // only if it starts inside its string's padded slot, 16-byte aligned; all loads are issued
    // before the first LDS write) and runs its rows
    const bool run = act && st == 0;
    bool running = run;
    for (int sub = 0; sub < K; sub += kContMaxRows) {
        if (__ballot(running) == 0) break;
        const int Ks = min(kContMaxRows, K - sub);
        int oA = 0, oB = 0, ib0 = 0;
        // the previous sub-block's LDS reads were issued before these writes (in order)
        if (running) {
            const uint8_t* pa = A + row;
            const uint8_t* pa0 = (const uint8_t*)((uintptr_t)pa & ~(uintptr_t)15);
            oA = (int)(pa - pa0);
            ib0 = max(row - a, 0);
            const uint8_t* pb = B + ib0;
            const uint8_t* pb0 = (const uint8_t*)((uintptr_t)pb & ~(uintptr_t)15);
            oB = (int)(pb - pb0);
            uint4 va[kStageA], vb[kStageB];
#pragma unroll
            for (int q = 0; q < kStageA; ++q)
                va[q] = (pa0 + 16 * q < A_end) ? reinterpret_cast<const uint4*>(pa0)[q] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int q = 0; q < kStageB; ++q)
                vb[q] = (pb0 + 16 * q < B_end) ? reinterpret_cast<const uint4*>(pb0)[q] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int q = 0; q < kStageA; ++q) {
                stage32[q * 256 + 0] = va[q].x; stage32[q * 256 + 1] = va[q].y;
                stage32[q * 256 + 2] = va[q].z; stage32[q * 256 + 3] = va[q].w;
            }
#pragma unroll
            for (int q = 0; q < kStageB; ++q) {
                const int o = (kStageA + q) * 256;
                stage32[o + 0] = vb[q].x; stage32[o + 1] = vb[q].y;
                stage32[o + 2] = vb[q].z; stage32[o + 3] = vb[q].w;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        {
            // every lane runs the rows of the sub-block, so the loop's control flow stays
            // wave-uniform (a lane's own exit would make the compiler copy the band and the
            // window at every row); a lane that is not running, or stops, computes rows whose
            // values are never used, and its reads stay inside its stage (ncs = 0: no column
            // byte is read)
            const int ncs = running ? nc : 0;
            // byte q of the lane's A blocks / B blocks (lane-interleaved 16-byte blocks)
            auto sa = [&](int q) -> int { return (int)stage8[((q >> 4) * 64) * 16 + (q & 15)]; };
            auto sb = [&](int ib) -> int {             // B[ib], 256 outside B
                const int q = oB + ib - ib0;
                return ((unsigned)ib < (unsigned)ncs)
                           ? (int)stage8[((kStageA + (q >> 4)) * 64) * 16 + (q & 15)] : 256;
            };
            // the window of rows r and r + 1: w[q] = B[rowstart + r - a + q], q <= MAXW (rows
            // taken in pairs, so the window shifts by two every second row)
            int w[MAXW + 1];
#pragma unroll
            for (int q = 0; q <= MAXW; ++q) w[q] = sb(row - a + q);
            const int rowstart = row;
            bool live = running;                       // the lane's rows still count
            // row r of the sub-block on the window w[O .. O + MAXW); false once no lane counts
            auto step = [&](int r, auto o) -> bool {
                constexpr int O = decltype(o)::value;
                const int ai = sa(oA + r);
                int left = BIG, emin = BIG;
#pragma unroll
                for (int q = 0; q < MAXW; ++q) {
                    const int up = (q + 1 < MAXW) ? M[(q + 1) < MAXW ? q + 1 : q] : BIG;
                    // min(up + 1, left + 1, diagonal + [mismatch]) as one three-way min of
                    // up, left and diagonal - [match], plus one
                    const int dm = M[q] - ((ai == w[q + O]) ? 1 : 0);
                    const int v = min(min(up, left), dm) + 1;
                    M[q] = v;
                    left = v;
                    const uint32_t ub = (uint32_t)b, uq = (uint32_t)q;
                    emin = min(emin, (int)(max(ub, uq) - min(ub, uq) + (uint32_t)v));
                }
                const int nrow = rowstart + r + 1;
                const bool fail = emin > t;            // Lemma 4: stop, return t + 1
                const bool last = nrow == nr;
                row = live ? nrow : row;
                // the final cell (band index b) only on a row where some lane ends
                int out = BIG;
                if (__ballot(live && !fail && last)) {
#pragma unroll
                    for (int q = 0; q < MAXW; ++q) out = (q == b) ? M[q] : out;
                }
                const int nst = fail ? 2 : last ? (out <= t ? 1 : 2) : 0;
                st = live ? nst : st;
                live = live && nst == 0;
                return __ballot(live) != 0;
            };
            for (int r = 0; r < Ks; r += 2) {
                if (!step(r, std::integral_constant<int, 0>{})) break;
                if (r + 1 >= Ks || !step(r + 1, std::integral_constant<int, 1>{})) break;
                if (r + 2 >= Ks) break;
#pragma unroll
                for (int q = 0; q + 1 < MAXW; ++q) w[q] = w[q + 2];
                w[MAXW - 1] = sb(rowstart - a + MAXW + r + 1);
                w[MAXW] = sb(rowstart - a + MAXW + r + 2);
            }
            running = st == 0;
        }
    }
    if (run && (st == 1 || st == 2)) my_cells += (uint64_t)band_cells(row, nc, a, b);
    append_tasks(run && st == 0, rec, cout + qbase, &cout_cnt[slot]);
    append_tasks(act && st == 1, rec, rout + qbase, &rout_cnt[slot]);
}

__global__ __launch_bounds__(64) void k_verify_first(VerifyParams V, Div div,
                                                     const LongRec* __restrict__ cands,
                                                     const uint32_t* __restrict__ slot_cnt,
                                                     const uint32_t* __restrict__ off, int K,
                                                     LongRec* __restrict__ cout, uint32_t* cout_cnt,
                                                     LongRec* __restrict__ rout, uint32_t* rout_cnt)
{
    __shared__ uint4 s_stage[(kStageA + kStageB) * 64];
    const int lane = threadIdx.x & 63;
    __attribute__((address_space(3))) uint32_t* stage =
        (__attribute__((address_space(3))) uint32_t*)s_stage + 4 * lane;
    uint64_t my_cells = 0, my_miss = 0;
    const SlotChunks S(slot_cnt, V.tau + 1, 64u);
    for (uint32_t ch = blockIdx.x; ch < S.total; ch += gridDim.x) {
        uint32_t b0, b1;
        const int slot = S.find(ch, &b0, &b1);
        const uint32_t base = off[slot];
#define PJ_FIRST(W) first_rows<W>(V, div, slot, cands + base, b0, b1, K, cout, cout_cnt, rout,     \
                                  rout_cnt, base, stage, my_cells, my_miss)
        if (slot + 1 <= 5) PJ_FIRST(5);
        else if (slot + 1 <= 9) PJ_FIRST(9);
        else if (slot + 1 <= 13) PJ_FIRST(13);
        else if (slot + 1 <= 17) PJ_FIRST(17);
        else if (slot + 1 <= 21) PJ_FIRST(21);
        else if (slot + 1 <= 25) PJ_FIRST(25);
        else if (slot + 1 <= 29) PJ_FIRST(29);
        else PJ_FIRST(33);
#undef PJ_FIRST
    }
    my_cells = wave_sum(my_cells);
    my_miss = wave_sum(my_miss);
    if (lane == 0) {
        unsigned long long* line = stat_line(V.counters, V.shards);
        if (my_cells) atomicAdd(&line[4], (unsigned long long)my_cells);
        if (my_miss) atomicAdd(&line[5], (unsigned long long)my_miss);
    }
}

// A part's DP by furthest rows (Ukkonen 1985; Landau and Vishkin 1989), L lanes a candidate and a band
// diagonal each: f(e, k) = the last row on diagonal k with distance up to e, found from the
// neighbours' rows at e - 1 and the characters that then agree, 32 at a time.  A diagonal is followed
// while e + |b - k| <= t, the cells the band's rows keep alive; a row passes Lemma 4's test exactly if
// some followed diagonal reaches it, so the rows the DP would have run, and its cells, are known
// without running them.  A part whose strings differ in d places costs d + 1 steps and a 32nd of its
// length.  Sets rows (run by the DP) and returns whether the part passes; the same in all L lanes.
struct __attribute__((packed)) Chars32 {
    uint64_t w[4];
};

template <int L>
__device__ inline bool far_part(const uint8_t* A, int nr, const uint8_t* B, int nc, int t, bool act,
                                int* rows)
{
    const int lane = threadIdx.x & 63, k = lane & (L - 1);
    constexpr int NONE = -(1 << 20);
    constexpr uint64_t kGroup = L == 64 ? ~0ull : (1ull << (L & 63)) - 1ull;
    const int delta = nc - nr, a = (t - delta) >> 1, b = (t + delta) >> 1;
    const int d = k - a, away = abs(b - k);
    const int lim = min(nr, nc - d);               // the diagonal's last row
    const bool in_band = k <= a + b;
    int f = NONE;
    bool done = !act || delta > t, pass = false;
    for (int e = 0; __ballot(!done) != 0; ++e) {
        const int from_left = __shfl_up(f, 1, L), from_right = __shfl_down(f, 1, L);
        const bool on = !done && in_band && e + away <= t;
        int row = e == 0 ? (d == 0 ? 0 : NONE)
                         : max(f + 1, max(k > 0 ? from_left : NONE, k < a + b ? from_right + 1 : NONE));
        row = min(row, lim);
        bool more = on && row >= 0 && row < lim;
        while (__ballot(more) != 0) {
            if (more) {
                const Chars32 u = *reinterpret_cast<const Chars32*>(A + row);
                const Chars32 v = *reinterpret_cast<const Chars32*>(B + row + d);
                int same = 32;
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    const uint64_t x = u.w[q] ^ v.w[q];
                    same = x ? 8 * q + (__builtin_ctzll(x) >> 3) : same;
                }
                row = min(row + same, lim);
                more = same == 32 && row < lim;
            }
        }
        if (on) f = row >= 0 ? row : NONE;
        const uint64_t ends = __ballot(on && k == b && f >= nr);
        if ((ends >> (lane & ~(L - 1))) & kGroup) pass = done = true;
        if (e >= t) done = true;
    }
    int far = in_band ? max(f, 0) : 0;
#pragma unroll
    for (int m = 1; m < L; m <<= 1) far = max(far, __shfl_xor(far, m, 64));
    *rows = pass ? nr : min(far + 1, nr);
    return pass;
}

// lanes a candidate: as many as a band of threshold t has diagonals, a power of two from 8
__device__ inline uint32_t far_lanes(int t) { return t < 8 ? 8u : t < 16 ? 16u : t < 32 ? 32u : 64u; }

// Side 0: the left parts that k_verify_first left; those that pass become right tasks.  Side 1: the
// right parts; those that pass are results.  A chunk is one slot's, so one threshold's.  In place of
// twelve more passes by rows, each with its queue of band rows: first rows and this, 10^5 long
// strings at tau = 16, 0.98 -> 0.30 ms; at tau = 32, where most candidates are not similar, 2.85 ->
// 2.3.  Bound by the latency of a step's two reads and two lane exchanges.
__global__ __launch_bounds__(kBlock) void k_verify_far(VerifyParams V, Div div, int side,
                                                       const LongRec* __restrict__ tasks,
                                                       const uint32_t* __restrict__ counts,
                                                       const uint32_t* __restrict__ off,
                                                       LongRec* __restrict__ rout,
                                                       uint32_t* rout_cnt)
{
    constexpr int kCap = 64;
    __shared__ uint64_t s_acc[kWaves][kCap];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    WaveAppender<uint64_t, kCap> acc{s_acc[w], 0};
    uint64_t my_cells = 0;
    auto threshold = [&](int slot) { return side == 0 ? slot : V.tau - slot; };
    const SlotChunks S(counts, V.tau + 1, 64u / far_lanes(max(threshold(lane), 0)));
    for (uint32_t ch = blockIdx.x * kWaves + (uint32_t)w; ch < S.total; ch += gridDim.x * kWaves) {
        uint32_t b0, b1;
        const int slot = __builtin_amdgcn_readfirstlane(S.find(ch, &b0, &b1));
        const int i = slot + 1, t = threshold(slot);
        const uint32_t lanes = far_lanes(t);
        const uint32_t k = b0 + (uint32_t)lane / lanes;
        const bool act = k < b1, first = ((uint32_t)lane & (lanes - 1)) == 0;
        // (groups past the end read the chunk's first task)
        const LongRec rec = tasks[off[slot] + (act ? k : b0)];
        const uint32_t meta = rec.a.z;
        const int p = (int)(meta & 2047u) + 1, l = (int)(meta >> 17), n = (int)rec.a.w;
        const uint8_t* x = V.x_arena + ((uint64_t)rec.b.y << 32 | rec.b.x);
        const uint8_t* y = V.y_arena + ((uint64_t)rec.b.w << 32 | rec.b.z);
        const Seg sg = partition_seg(l, i, V.tau, div);
        const int ry = sg.p - 1 + sg.len, rx = p - 1 + sg.len;
        const uint8_t* r = side == 0 ? y : y + ry;
        const uint8_t* s = side == 0 ? x : x + rx;
        const int lr = side == 0 ? sg.p - 1 : l - ry, ls = side == 0 ? p - 1 : n - rx;
        const bool yrows = lr <= ls;
        const uint8_t* A = yrows ? r : s;
        const uint8_t* B = yrows ? s : r;
        const int nr = yrows ? lr : ls, nc = yrows ? ls : lr, delta = nc - nr;
        int rows = 0;
        bool pass;
        if (lanes == 8) pass = far_part<8>(A, nr, B, nc, t, act, &rows);
        else if (lanes == 16) pass = far_part<16>(A, nr, B, nc, t, act, &rows);
        else if (lanes == 32) pass = far_part<32>(A, nr, B, nc, t, act, &rows);
        else pass = far_part<64>(A, nr, B, nc, t, act, &rows);
        if (act && first && delta <= t)
            my_cells += (uint64_t)band_cells(rows, nc, (t - delta) >> 1, (t + delta) >> 1);
        if (side == 0) append_tasks(pass && first, rec, rout + off[slot], &rout_cnt[slot]);
        else acc.push(pass && first, (uint64_t)rec.a.x << 32 | rec.a.y, V.out, V.out_cap,
                      &V.counters[3]);
    }
    block_flush(acc, V.out, V.out_cap, &V.counters[3]);
    block_add(&stat_line(V.counters, V.shards)[4], my_cells);
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, int n, uint32_t v)
{
    for (int k = threadIdx.x; k < n; k += blockDim.x) p[k] = v;
}

template <int MAXW>
__global__ __launch_bounds__(kBlock) void k_short(const uint8_t* __restrict__ x_arena,
                                                  const uint16_t* __restrict__ x_slen,
                                                  const int32_t* __restrict__ x_lenstart,
                                                  const int64_t* __restrict__ x_gbase,
                                                  int x_lmax,
                                                  const uint8_t* __restrict__ y_arena,
                                                  const uint16_t* __restrict__ y_slen,
                                                  const int32_t* __restrict__ y_lenstart,
                                                  const int64_t* __restrict__ y_gbase,
                                                  uint32_t y_first, uint32_t y_count, int tau,
                                                  int self, const int32_t* __restrict__ q_tau,
                                                  uint64_t* __restrict__ out,
                                                  uint64_t out_cap, int shards,
                                                  unsigned long long* __restrict__ counters)
{
    const int lane = threadIdx.x & 63;
    uint64_t examined = 0;
    for (uint32_t yi = blockIdx.x; yi < y_count; yi += gridDim.x) {
        const uint32_t gy = y_first + yi;
        const int ly = y_slen[gy];
        const uint8_t* y = y_arena + y_gbase[ly] + (int64_t)(gy - y_lenstart[ly]) * stride_of(ly);
        const int lo_len = ly - tau < 0 ? 0 : ly - tau;
        int hi_len = ly + tau;
        if (hi_len > x_lmax) hi_len = x_lmax;
        if (hi_len < lo_len) continue;
        const uint32_t g0 = (uint32_t)x_lenstart[lo_len], g1 = (uint32_t)x_lenstart[hi_len + 1];
        for (uint32_t base = g0; base < g1; base += kBlock) {
            uint32_t gx = base + threadIdx.x;
            bool pass = false;
            if (gx < g1) {
                const int lx = x_slen[gx];
                const int tx = q_tau ? q_tau[gx] : tau;      // the pair's threshold
                const int dlen = lx > ly ? lx - ly : ly - lx;
                bool take = ly <= tx && dlen <= tx && !(self && lx <= tau && gx >= gy);
                if (take) {
                    const uint8_t* x = x_arena + x_gbase[lx] +
                                       (int64_t)(gx - x_lenstart[lx]) * stride_of(lx);
                    int c = 0;
                    pass = vsp_global<MAXW>(y, ly, x, lx, tx, &c) <= tx;
                    examined += 1;
                }
            }
            uint64_t pm = __ballot(pass);
            if (pm) {
                int leader = __ffsll((unsigned long long)pm) - 1;
                unsigned long long b = 0;
                if (lane == leader) b = atomicAdd(&counters[3], (unsigned long long)__popcll(pm));
                b = __shfl(b, leader, 64);
                if (pass) {
                    uint64_t idx = b + (uint64_t)__popcll(pm & lanemask_lt());
                    if (idx < out_cap) out[idx] = ((uint64_t)gx << 32) | gy;
                }
            }
        }
    }
    block_add(&stat_line(counters, shards)[6], examined);
}

// ------------------------------------------------------------------------------------------
// Output: map accepted (gx, gy) to ids, sort, deduplicate (the result is a set, Algorithm 1)
// ------------------------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_pairs_to_keys(const uint64_t* __restrict__ acc,
                                                          uint64_t m,
                                                          const int32_t* __restrict__ xperm,
                                                          const int32_t* __restrict__ yperm,
                                                          int self, int bbits,
                                                          uint64_t* __restrict__ keys)
{
    uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= m) return;
    uint64_t v = acc[k];
    uint32_t a = (uint32_t)xperm[v >> 32];
    uint32_t b = (uint32_t)yperm[v & 0xffffffffu];
    if (self && b < a) { uint32_t t = a; a = b; b = t; }
    keys[k] = ((uint64_t)a << bbits) | b;
}

// out[g] = in[perm[g]]: per-id values (a query's tau) moved to sorted positions.
__global__ __launch_bounds__(kBlock) void k_gather_i32(const int32_t* __restrict__ in,
                                                       const int32_t* __restrict__ perm, int64_t n,
                                                       int32_t* __restrict__ out)
{
    int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (g < n) out[g] = in[perm[g]];
}

// ------------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------------

static inline unsigned blocks_for(uint64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

hipError_t launch_length_hist(const int32_t* offs, int64_t n, int32_t* lcount, int32_t* lenstart,
                              int64_t* gbase, uint32_t* bitmap, uint16_t* code, hipStream_t s)
{
    if ((bitmap == nullptr) != (code == nullptr)) return hipErrorInvalidValue;
    // a block also for no strings: the tables are always written
    const unsigned grid =
        (unsigned)std::min<uint64_t>(((uint64_t)n + kBlock - 1) / kBlock, 256);
    if (grid > 0)
        hipLaunchKernelGGL(k_length_hist, dim3(grid), dim3(kBlock), 0, s, offs, n, lcount);
    hipLaunchKernelGGL(k_length_tables, dim3(1), dim3(kBlock), 0, s, lcount, lenstart, gbase, bitmap,
                       code);
    return hipGetLastError();
}

hipError_t launch_iota_len_keys(const int32_t* offs, int64_t n, uint32_t* keys, uint32_t* vals,
                                hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_len_keys, dim3(blocks_for(n)), dim3(kBlock), 0, s, offs, n, keys, vals);
    return hipGetLastError();
}

hipError_t launch_pack_arena(const uint8_t* bytes, const int32_t* offs, const int32_t* perm,
                             int64_t n, const int32_t* lenstart, const int64_t* gbase,
                             uint8_t* sarena, uint16_t* slen, int lmax, uint32_t* bitmap,
                             hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    // lanes for the widest slot, up to a wave
    int lps_shift = 0;
    while (lps_shift < 6 && (16 << lps_shift) < lmax) ++lps_shift;
    const uint64_t threads = (uint64_t)n << lps_shift;
    const uint64_t blocks = std::min<uint64_t>((threads + kBlock - 1) / kBlock, bitmap ? 2048 : 65536);
    hipLaunchKernelGGL(k_pack_arena, dim3((unsigned)blocks), dim3(kBlock), 0, s, bytes, offs, perm,
                       n, lenstart, gbase, sarena, slen, lps_shift, bitmap);
    return hipGetLastError();
}

hipError_t launch_emit_segments(const DevSet& S, int tau, int64_t g_first, int64_t g_count,
                                int64_t* inl_base, uint64_t* keys, uint32_t* vals, hipStream_t s)
{
    if (g_count <= 0) return hipSuccess;
    if (!S.bitmap || !S.code) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_emit_segments, dim3(blocks_for((uint64_t)g_count * (uint64_t)(tau + 1))),
                       dim3(kBlock), 0, s, S.sarena, S.slen, S.lenstart, S.gbase, tau, g_first,
                       g_count, make_div(tau + 1), S.bitmap, S.code, inl_base, keys, vals);
    return hipGetLastError();
}

hipError_t launch_gather_inline(const DevSet& S, const uint64_t* keys, const uint32_t* vals,
                                int64_t E, int tau, const int64_t* inl_base, uint8_t* inl,
                                hipStream_t s)
{
    if (E <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_inline, dim3(blocks_for(E)), dim3(kBlock), 0, s, keys, vals, E,
                       tau, S.sarena, S.lenstart, S.gbase, inl_base, inl);
    return hipGetLastError();
}

hipError_t launch_list_dir(const uint64_t* keys, const uint32_t* runstart, uint32_t nruns, uint32_t E,
                           uint32_t ngroups, uint32_t* bounds, uint32_t* words, void* scan_tmp,
                           size_t scan_bytes, uint4* recs, uint32_t* gdir, uint2* dir,
                           hipStream_t s)
{
    if (ngroups == 0 || nruns == 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_list_records, dim3(blocks_for((uint64_t)nruns + 1)), dim3(kBlock), 0, s,
                       keys, runstart, nruns, E, ngroups, recs, bounds);
    hipLaunchKernelGGL(k_dir_words, dim3(blocks_for(ngroups)), dim3(kBlock), 0, s, bounds, ngroups,
                       words);
    hipError_t e = scan_u32_to_u32(words, gdir, ngroups, scan_tmp, scan_bytes, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dir_fill, dim3(blocks_for(nruns)), dim3(kBlock), 0, s, recs, nruns, gdir,
                       dir);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_hit_counts(const Hit* __restrict__ hits, uint64_t nh,
                                                       uint32_t* __restrict__ counts)
{
    uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k < nh) counts[k] = hits[k].count;
}

hipError_t launch_hit_counts(const Hit* hits, uint64_t nh, uint32_t* counts, hipStream_t s)
{
    if (nh == 0) return hipSuccess;
    hipLaunchKernelGGL(k_hit_counts, dim3(blocks_for(nh)), dim3(kBlock), 0, s, hits, nh, counts);
    return hipGetLastError();
}

// Multi-match window size of slot i for a length difference delta = n - l (Sec. 4.2: the
// start positions p_i - (i-1) .. p_i + (i-1) intersected with p_i + delta - (tau+1-i) ..
// p_i + delta + (tau+1-i)), 0 when empty
__device__ inline int mm_window_size(int tau, int i, int delta)
{
    const int r = tau + 1 - i;
    const int a = (i - 1) < delta + r ? (i - 1) : delta + r;
    const int b = (i - 1) < r - delta ? (i - 1) : r - delta;
    const int sz = a + b + 1;
    return sz > 0 ? sz : 0;
}

// One block: the (length, slot) pairs of a probe string grouped by decreasing window size
// (a counting sort on the size; the order within a size is whatever the atomics give).  Pairs
// of one size take equally many steps of the probe's window walk, so a wave whose lanes hold
// them keeps all its lanes busy.
__global__ __launch_bounds__(kBlock) void k_probe_order(int tau, int nl, int self,
                                                        uint16_t* __restrict__ order)
{
    constexpr int kSizes = 2 * kTauMax + 2;      // window sizes 0 .. 2 tau + 1
    __shared__ uint32_t cnt[kSizes];
    const int T1 = tau + 1, per = nl * T1;
    auto size_of = [&](int r) {
        const int dl = r / T1, i = r % T1 + 1;
        return mm_window_size(tau, i, self ? dl : tau - dl);
    };
    for (int k = threadIdx.x; k < kSizes; k += kBlock) cnt[k] = 0;
    __syncthreads();
    for (int r = threadIdx.x; r < per; r += kBlock) atomicAdd(&cnt[size_of(r)], 1u);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int k = kSizes - 1; k >= 0; --k) {
            const uint32_t c = cnt[k];
            cnt[k] = run;
            run += c;
        }
    }
    __syncthreads();
    for (int r = threadIdx.x; r < per; r += kBlock)
        order[atomicAdd(&cnt[size_of(r)], 1u)] = (uint16_t)r;
}

// One block: the item list.  Thread t lays down the windows of its run of consecutive pairs.
__global__ __launch_bounds__(kBlock) void k_probe_items(int tau, int nl, int self,
                                                        uint32_t* __restrict__ items,
                                                        uint32_t* __restrict__ chunk)
{
    __shared__ uint32_t s_wave[kWaves];
    const int T1 = tau + 1, pairs = nl * T1;
    const int per = (pairs + kBlock - 1) / kBlock;
    const int r0 = min((int)threadIdx.x * per, pairs), r1 = min(r0 + per, pairs);
    auto size_of = [&](int r) {
        const int dl = r / T1, i = r % T1 + 1;
        return (uint32_t)mm_window_size(tau, i, self ? dl : tau - dl);
    };
    uint32_t mine = 0;
    for (int r = r0; r < r1; ++r) mine += size_of(r);
    uint32_t total;
    uint32_t at = block_excl_scan<uint32_t>(mine, s_wave, &total);
    for (int r = r0; r < r1; ++r) {
        if (r % kItemPairs == 0) chunk[r / kItemPairs] = at;
        const uint32_t sz = size_of(r);
        for (uint32_t s = 0; s < sz; ++s) items[at + s] = (uint32_t)r << 8 | s;
        at += sz;
    }
    if (threadIdx.x == 0) chunk[(pairs + kItemPairs - 1) / kItemPairs] = total;
}

uint64_t probe_item_count(int tau, int nl, int self)
{
    // Lemma 2 for each length difference
    uint64_t n = 0;
    for (int dl = 0; dl < nl; ++dl) {
        const int d = self ? dl : tau - dl;
        n += (uint64_t)((tau * tau - d * d) / 2 + tau + 1);
    }
    return n;
}

hipError_t launch_probe_items(int tau, int nl, int self, uint32_t* items, uint32_t* chunk,
                              hipStream_t s)
{
    if (tau < 0 || tau > kTauMax || nl < 1 || nl > 2 * kTauMax + 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_probe_items, dim3(1), dim3(kBlock), 0, s, tau, nl, self, items, chunk);
    return hipGetLastError();
}

hipError_t launch_probe_order(int tau, int nl, int self, uint16_t* order, hipStream_t s)
{
    if (tau < 0 || tau > kTauMax || nl < 1 || nl > 2 * kTauMax + 1 || !order)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_probe_order, dim3(1), dim3(kBlock), 0, s, tau, nl, self, order);
    return hipGetLastError();
}

hipError_t launch_probe(const ProbeParams& P, int max_blocks, hipStream_t s)
{
    if (P.threads == 0) return hipSuccess;
    if (!P.sym.code) return hipErrorInvalidValue;
    const uint64_t blocks = std::min<uint64_t>(blocks_for(P.threads), (uint64_t)max_blocks);
    hipLaunchKernelGGL(k_probe, dim3((unsigned)blocks), dim3(kBlock), 0, s, P, make_div(P.tau + 1));
    return hipGetLastError();
}

hipError_t launch_probe_tiles(const ProbeParams& P, const ProbeTiles& T, int max_blocks,
                              hipStream_t s)
{
    if (T.tiles == 0) return hipSuccess;
    if (!P.sym.code || P.q_tau || P.nx_dev || T.groups < 1 || T.maxlen > kTileMaxLen ||
        (uint64_t)T.tiles * T.groups > 0x7fffffffull)
        return hipErrorInvalidValue;
    const uint64_t units = (uint64_t)T.tiles * T.groups;
    // a multiple of the XCDs
    const dim3 grid((unsigned)std::min<uint64_t>(((units + kWaves - 1) / kWaves + 7) / 8 * 8,
                                                 (uint64_t)std::max(max_blocks / 8 * 8, 8)));
    const Div div = make_div(P.tau + 1);
#define PJ_TILES(MAXQ, HITS)                                                                       \
    hipLaunchKernelGGL((k_probe_tiles<MAXQ, HITS>), grid, dim3(kBlock), 0, s, P, div, T)
    const bool many = P.tau >= 2;              // hits: see the kernel
    if (T.maxlen <= 32) { if (many) PJ_TILES(2, 512); else PJ_TILES(2, 256); }
    else if (T.maxlen <= 64) { if (many) PJ_TILES(4, 512); else PJ_TILES(4, 256); }
    else PJ_TILES(8, 256);
#undef PJ_TILES
    return hipGetLastError();
}

hipError_t launch_probe_long(const ProbeParams& P, const ProbeItems& I, uint32_t g_first,
                             uint32_t g_end, int maxlen, int max_blocks, hipStream_t s)
{
    if (g_first >= g_end) return hipSuccess;
    if (!P.sym.code || P.q_tau || P.nx_dev || P.selection != 0 || !I.items ||
        I.chunks != (P.nl * (P.tau + 1) + kItemPairs - 1) / kItemPairs)
        return hipErrorInvalidValue;
    const dim3 grid(std::min<unsigned>(g_end - g_first, (unsigned)max_blocks));
    const Div div = make_div(P.tau + 1);
    if (maxlen < 1024)
        hipLaunchKernelGGL(k_probe_long<1024>, grid, dim3(kBlock), 0, s, P, div, I, g_first, g_end);
    else
        hipLaunchKernelGGL(k_probe_long<2048>, grid, dim3(kBlock), 0, s, P, div, I, g_first, g_end);
    return hipGetLastError();
}

template <int W>
static void verify_w(const VerifyParams& V, int grid, hipStream_t s)
{
    hipLaunchKernelGGL((k_verify<W>), dim3(grid), dim3(kBlock), 0, s, V, make_div(V.tau + 1));
}

template <int W>
static void verify_batched_w(const VerifyParams& V, const uint32_t* first, uint64_t nchunks,
                             int grid, hipStream_t s)
{
    if (W == 9 && V.tau >= 6 && V.tau <= 8 && V.y_maxlen <= 40)
        hipLaunchKernelGGL((k_verify_batched<W, (W == 9 ? 2 : 0)>), dim3(grid), dim3(kBlock), 0,
                           s, V, make_div(V.tau + 1), first, nchunks);
    else if (W == 9 && V.tau <= 8 && V.y_maxlen <= kStgY - 4)
        hipLaunchKernelGGL((k_verify_batched<W, (W == 9 ? 1 : 0)>), dim3(grid), dim3(kBlock), 0,
                           s, V, make_div(V.tau + 1), first, nchunks);
    else
        hipLaunchKernelGGL((k_verify_batched<W, 0>), dim3(grid), dim3(kBlock), 0, s, V,
                           make_div(V.tau + 1), first, nchunks);
}

uint64_t batched_chunks(uint64_t ncand, int rounds)
{
    const uint64_t chunk = 64ull * (uint64_t)rounds;
    return (ncand + chunk - 1) / chunk;
}

unsigned slot_bucket_grid(uint64_t nh_cap)
{
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((nh_cap + kBlock - 1) / kBlock, 2048));
}

hipError_t launch_slot_bucket(const Hit* hits, const unsigned long long* nh_dev, uint64_t nh_cap,
                              uint32_t big, uint32_t* bb, uint32_t* bb_off, void* scan_tmp,
                              size_t scan_bytes, Hit* out, hipStream_t s)
{
    if (nh_cap == 0) return hipSuccess;
    const unsigned grid = slot_bucket_grid(nh_cap);
    hipLaunchKernelGGL(k_slot_hist, dim3(grid), dim3(kBlock), 0, s, hits, nh_dev, big, bb);
    hipError_t e = scan_u32_to_u32(bb, bb_off, (uint64_t)grid * kHitBuckets, scan_tmp, scan_bytes,
                                   s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_slot_scatter, dim3(grid), dim3(kBlock), 0, s, hits, nh_dev, big, bb_off,
                       out);
    return hipGetLastError();
}

template <int W, int NC>
static void verify_segs_wn(const VerifyParams& V, const Hit* big, const uint32_t* segp,
                           uint64_t nbig, uint64_t nseg, const uint32_t* first, uint64_t nchunks,
                           uint32_t chunk, int grid, unsigned long long* ticket, hipStream_t s)
{
    // one candidate per lane with strings of at most 40 bytes: 44-byte lane slots
    if (NC == 1 && W == 9 && V.y_maxlen <= 40)
        hipLaunchKernelGGL((k_verify_segs<W, (NC == 1 && W == 9) ? 40 : 48, NC>), dim3(grid),
                           dim3(kBlock), 0, s, V, make_div(V.tau + 1), big, segp, nbig, nseg,
                           first, nchunks, chunk, ticket);
    else if (V.y_maxlen <= 48)
        hipLaunchKernelGGL((k_verify_segs<W, 48, NC>), dim3(grid), dim3(kBlock), 0, s, V,
                           make_div(V.tau + 1), big, segp, nbig, nseg, first, nchunks, chunk, ticket);
    else if (V.y_maxlen <= 64)
        hipLaunchKernelGGL((k_verify_segs<W, 64, NC>), dim3(grid), dim3(kBlock), 0, s, V,
                           make_div(V.tau + 1), big, segp, nbig, nseg, first, nchunks, chunk, ticket);
    else
        hipLaunchKernelGGL((k_verify_segs<W, 0, 1>), dim3(grid), dim3(kBlock), 0, s, V,
                           make_div(V.tau + 1), big, segp, nbig, nseg, first, nchunks, chunk, ticket);
}

template <int W>
static void verify_segs_w(const VerifyParams& V, const Hit* big, const uint32_t* segp,
                          uint64_t nbig, uint64_t nseg, const uint32_t* first, uint64_t nchunks,
                          uint32_t chunk, int lane_cands, int grid, unsigned long long* ticket,
                          hipStream_t s)
{
    if constexpr (W <= 9) {
        if (lane_cands == 2) {
            verify_segs_wn<W, 2>(V, big, segp, nbig, nseg, first, nchunks, chunk, grid, ticket, s);
            return;
        }
    }
    verify_segs_wn<W, 1>(V, big, segp, nbig, nseg, first, nchunks, chunk, grid, ticket, s);
}

uint64_t seg_chunks(uint64_t nseg, int chunk) { return (nseg + (uint64_t)chunk - 1) / (uint64_t)chunk; }

// members per list segment: 64 per candidate a lane takes (two per lane only when the indexed
// strings fit in registers and the band is at most 9 wide)
int seg_members(int y_maxlen, int tau, int lane_cands)
{
    return (lane_cands == 2 && y_maxlen <= 64 && tau + 1 <= 9) ? 128 : 64;
}

hipError_t launch_seg_counts(const Hit* big, uint64_t nbig, int members, uint32_t* segs,
                             hipStream_t s)
{
    if (nbig == 0) return hipSuccess;
    hipLaunchKernelGGL(k_seg_counts, dim3(blocks_for(nbig)), dim3(kBlock), 0, s, big, nbig,
                       (uint32_t)members, segs);
    return hipGetLastError();
}

hipError_t launch_verify_segs(const VerifyParams& V, const Hit* big, const uint32_t* segp,
                              uint64_t nbig, uint64_t nseg, uint32_t* first, int chunk,
                              int lane_cands, int grid, unsigned long long* ticket, hipStream_t s)
{
    if (nbig == 0 || nseg == 0) return hipSuccess;
    if (chunk < 1 || grid < 1 || lane_cands < 1 || lane_cands > 2) return hipErrorInvalidValue;
    const uint64_t nchunks = seg_chunks(nseg, chunk);
    const uint32_t c = (uint32_t)chunk;
    hipLaunchKernelGGL(k_seg_chunk_starts, dim3(blocks_for(nchunks)), dim3(kBlock), 0, s, segp,
                       nbig, nchunks, c, first);
    const int w = V.tau + 1;
    const int lc = lane_cands;
    if (w <= 5 && lc == 1 && V.y_maxlen <= kAutoMaxLen)
        return launch_verify_auto(V, big, nbig, segp, nseg, first, nchunks, c, (uint64_t)grid * kWaves,
                                  ticket, s);
    if (w <= 5) verify_segs_w<5>(V, big, segp, nbig, nseg, first, nchunks, c, lc, grid, ticket, s);
    else if (w <= 9) verify_segs_w<9>(V, big, segp, nbig, nseg, first, nchunks, c, lc, grid, ticket, s);
    else if (w <= 17) verify_segs_w<17>(V, big, segp, nbig, nseg, first, nchunks, c, lc, grid, ticket, s);
    else if (w <= 33) verify_segs_w<33>(V, big, segp, nbig, nseg, first, nchunks, c, lc, grid, ticket, s);
    else verify_segs_w<64>(V, big, segp, nbig, nseg, first, nchunks, c, lc, grid, ticket, s);
    return hipGetLastError();
}

hipError_t launch_chain_counts(const Hit* big, uint64_t nbig, const uint16_t* x_slen,
                               const uint32_t* runlen, int self, uint32_t* chains, hipStream_t s)
{
    if (nbig == 0) return hipSuccess;
    hipLaunchKernelGGL(k_chain_counts, dim3(blocks_for(nbig)), dim3(kBlock), 0, s, big, nbig,
                       x_slen, runlen, self, chains);
    return hipGetLastError();
}

hipError_t launch_verify_chains(const VerifyParams& V, const Hit* big,
                                const unsigned long long* cprefix, uint64_t nbig,
                                uint64_t nchains, uint32_t* first, int grid, hipStream_t s)
{
    if (nbig == 0 || nchains == 0) return hipSuccess;
    if (grid < 1 || V.tau + 1 > kShareMaxW || !V.svals || !V.runlen) return hipErrorInvalidValue;
    const uint64_t nchunks = (nchains + 63) / 64;
    hipLaunchKernelGGL(k_chunk_starts, dim3(blocks_for(nchunks)), dim3(kBlock), 0, s, cprefix,
                       nbig, nchunks, 64ull, first);
    const Div div = make_div(V.tau + 1);
    if (V.tau + 1 <= 5)
        hipLaunchKernelGGL((k_verify_chains<5>), dim3(grid), dim3(kBlock), 0, s, V, div, big,
                           cprefix, nbig, nchains, first, nchunks);
    else
        hipLaunchKernelGGL((k_verify_chains<9>), dim3(grid), dim3(kBlock), 0, s, V, div, big,
                           cprefix, nbig, nchains, first, nchunks);
    return hipGetLastError();
}

hipError_t launch_prefix8_keys(const DevSet& S, const uint32_t* vals, int64_t E, uint64_t* keys,
                               uint32_t* idx, hipStream_t s)
{
    if (E == 0) return hipSuccess;
    hipLaunchKernelGGL(k_prefix8_keys, dim3(blocks_for((uint64_t)E)), dim3(kBlock), 0, s, vals,
                       E, S.sarena, S.slen, S.lenstart, S.gbase, keys, idx);
    return hipGetLastError();
}

hipError_t launch_gather_keys(const uint64_t* keys, const uint32_t* idx, int64_t E,
                              uint64_t* out, hipStream_t s)
{
    if (E == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_keys, dim3(blocks_for((uint64_t)E)), dim3(kBlock), 0, s, keys,
                       idx, E, out);
    return hipGetLastError();
}

hipError_t launch_gather_vals(const uint32_t* vals, const uint32_t* idx, int64_t E, uint32_t* out,
                              hipStream_t s)
{
    if (E == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_vals, dim3(blocks_for((uint64_t)E)), dim3(kBlock), 0, s, vals,
                       idx, E, out);
    return hipGetLastError();
}

hipError_t launch_run_lengths(const uint32_t* runstart, uint32_t nruns, uint32_t E,
                              uint32_t* runlen, hipStream_t s)
{
    if (nruns == 0) return hipSuccess;
    hipLaunchKernelGGL(k_run_lengths, dim3(blocks_for(nruns)), dim3(kBlock), 0, s, runstart,
                       nruns, E, runlen);
    return hipGetLastError();
}

// count arrays of 256 u32: slot counts, offsets, cursors, right tasks, left tasks not done
constexpr int kLongCounts = 5;

size_t long_scratch_bytes(uint64_t ncand)
{
    const uint64_t rc = (ncand * sizeof(LongRec) + 255) & ~(uint64_t)255;
    // candidates, right tasks, left tasks not done
    return kLongCounts * 256 * sizeof(uint32_t) + 3 * rc;
}

hipError_t launch_verify_long(const VerifyParams& V, uint64_t ncand, void* scratch, int grid,
                              hipStream_t s)
{
    if (V.nhits == 0 || ncand == 0) return hipSuccess;
    if (V.tau + 1 > kContW || grid < 1 || V.q_tau) return hipErrorInvalidValue;
    uint8_t* p = (uint8_t*)scratch;
    uint32_t* slot_cnt = (uint32_t*)p;
    uint32_t* off = slot_cnt + 256;
    uint32_t* cursor = off + 256;
    uint32_t* right_cnt = cursor + 256;
    uint32_t* left_cnt = right_cnt + 256;
    const uint64_t rc = (ncand * sizeof(LongRec) + 255) & ~(uint64_t)255;
    uint8_t* q = p + kLongCounts * 256 * sizeof(uint32_t);
    LongRec* cands = (LongRec*)q;
    LongRec* right = (LongRec*)(q + rc);
    LongRec* left = (LongRec*)(q + 2 * rc);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, s, slot_cnt, kLongCounts * 256, 0u);
    const unsigned hb = (unsigned)std::min<uint64_t>(blocks_for(V.nhits), 4096);
    hipLaunchKernelGGL(k_long_slot_counts, dim3(hb), dim3(kBlock), 0, s, V.hits, V.nhits, slot_cnt);
    hipLaunchKernelGGL(k_long_slot_offsets, dim3(1), dim3(64), 0, s, slot_cnt, off, cursor);
    hipLaunchKernelGGL(k_long_scatter, dim3(hb), dim3(kBlock), 0, s, V.hits,
                       V.nhits, V.vals, V.x_slen, V.x_lenstart, V.x_gbase, V.y_lenstart,
                       V.y_gbase, cursor, cands);
    const Div div = make_div(V.tau + 1);
    // rows of the first pass (10^5 long strings, ms in all with 16 / 32 / 64: tau = 8 0.16, 0.16,
    // 0.17; 16 0.30, 0.30, 0.31; 24 0.81, 0.77, 0.79; 32 2.88, 2.28, 2.41); PJ_LONG_PASSES sets
    // them (tests and tuning; it changes no result): the first of a comma list of row counts
    int K = 32;
    if (const char* e = getenv("PJ_LONG_PASSES")) {
        for (const char* c = e; *c;) {
            const int v = atoi(c);
            if (v < 1 || v > 4096) return hipErrorInvalidValue;
            if (c == e) K = v;
            while (*c && *c != ',') ++c;
            if (*c == ',') ++c;
        }
    }
    hipLaunchKernelGGL(k_verify_first, dim3(grid), dim3(64), 0, s, V, div, cands, slot_cnt, off, K,
                       left, left_cnt, right, right_cnt);
    hipLaunchKernelGGL(k_verify_far, dim3(grid), dim3(kBlock), 0, s, V, div, 0, left, left_cnt, off,
                       right, right_cnt);
    hipLaunchKernelGGL(k_verify_far, dim3(grid), dim3(kBlock), 0, s, V, div, 1, right, right_cnt, off,
                       (LongRec*)nullptr, (uint32_t*)nullptr);
    return hipGetLastError();
}

hipError_t launch_verify_batched(const VerifyParams& V, uint32_t* first, int grid, hipStream_t s)
{
    if (V.ncand == 0) return hipSuccess;
    if (V.wave_rounds < 1 || V.wave_rounds > kWaveRounds) return hipErrorInvalidValue;
    const uint64_t nchunks = batched_chunks(V.ncand, V.wave_rounds);
    hipLaunchKernelGGL(k_chunk_starts, dim3(blocks_for(nchunks)), dim3(kBlock), 0, s, V.prefix,
                       V.nhits, nchunks, 64ull * (uint64_t)V.wave_rounds, first);
    const int w = V.tau + 1;
    if (w <= 9) verify_batched_w<9>(V, first, nchunks, grid, s);
    else if (w <= 17) verify_batched_w<17>(V, first, nchunks, grid, s);
    else if (w <= 33) verify_batched_w<33>(V, first, nchunks, grid, s);
    else verify_batched_w<64>(V, first, nchunks, grid, s);
    return hipGetLastError();
}

hipError_t launch_verify(const VerifyParams& V, int grid, hipStream_t s)
{
    if (V.ncand == 0) return hipSuccess;
    const int w = V.tau + 1;
    if (w <= 2) verify_w<2>(V, grid, s);
    else if (w <= 3) verify_w<3>(V, grid, s);
    else if (w <= 5) verify_w<5>(V, grid, s);
    else if (w <= 9) verify_w<9>(V, grid, s);
    else if (w <= 17) verify_w<17>(V, grid, s);
    else if (w <= 33) verify_w<33>(V, grid, s);
    else verify_w<64>(V, grid, s);
    return hipGetLastError();
}

template <int W>
static void short_w(const DevSet& P, const DevSet& Y, int tau, int self, const int32_t* q_tau,
                    uint32_t y_first, uint32_t y_count, uint64_t* out, uint64_t cap,
                    unsigned long long* ctr, hipStream_t s)
{
    unsigned grid = y_count < 65536 ? y_count : 65536;
    hipLaunchKernelGGL((k_short<W>), dim3(grid), dim3(kBlock), 0, s, P.sarena, P.slen, P.lenstart,
                       P.gbase, P.lmax, Y.sarena, Y.slen, Y.lenstart, Y.gbase, y_first, y_count,
                       tau, self, q_tau, out, cap, kStatShards, ctr);
}

hipError_t launch_short_path(const DevSet& P, const DevSet& Y, int tau, int self,
                             const int32_t* q_tau, uint64_t* out, uint64_t out_cap,
                             unsigned long long* counters, hipStream_t s)
{
    if (Y.n == 0 || P.n == 0 || Y.lmin > tau) return hipSuccess;
    const int top = tau < Y.lmax ? tau : Y.lmax;
    uint32_t y_first = (uint32_t)Y.h_lenstart[0];
    uint32_t y_end = (uint32_t)Y.h_lenstart[top + 1];
    if (y_end <= y_first) return hipSuccess;
    uint32_t cnt = y_end - y_first;
    const int w = tau + 1;
    if (w <= 2) short_w<2>(P, Y, tau, self, q_tau, y_first, cnt, out, out_cap, counters, s);
    else if (w <= 5) short_w<5>(P, Y, tau, self, q_tau, y_first, cnt, out, out_cap, counters, s);
    else if (w <= 9) short_w<9>(P, Y, tau, self, q_tau, y_first, cnt, out, out_cap, counters, s);
    else if (w <= 17) short_w<17>(P, Y, tau, self, q_tau, y_first, cnt, out, out_cap, counters, s);
    else if (w <= 33) short_w<33>(P, Y, tau, self, q_tau, y_first, cnt, out, out_cap, counters, s);
    else short_w<64>(P, Y, tau, self, q_tau, y_first, cnt, out, out_cap, counters, s);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Captured query batches: the sizes of a batch live in device memory, so one instantiated graph
// of these launches serves every batch of a serving slot.
// ------------------------------------------------------------------------------------------

// One block: exclusive prefix of the hits' candidate counts, the batch's sizes, and first[ch] (the
// hit holding candidate ch * chunk: a hit writes the chunks that begin inside it).  A chunk is a
// wave's 64 candidates until every wave of a full chip has one, then more rounds of 64.  An
// overflow (more hits than the buffer holds, or more candidates than the batch may have) sets a
// flag and leaves nothing to verify; the host then runs the batch another way.
__global__ __launch_bounds__(1024) void k_batch_prefix(const Hit* __restrict__ hits,
                                                       const unsigned long long* __restrict__ counters,
                                                       uint64_t hit_cap,
                                                       unsigned long long* __restrict__ prefix,
                                                       unsigned long long* __restrict__ bc,
                                                       uint32_t* __restrict__ first,
                                                       uint64_t cand_cap)
{
    constexpr int PER = 4;
    __shared__ unsigned long long s_w[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t nh = counters[0], ncand = counters[1];
    unsigned long long flags = 0;
    if (nh > hit_cap) flags |= 1;
    if (ncand > cand_cap) flags |= 2;
    if (flags) nh = ncand = 0;
    const uint64_t per_wave = (ncand + 64ull * kBatchWaves - 1) / (64ull * kBatchWaves);
    const uint64_t rounds = per_wave < 1 ? 1 : per_wave > kWaveRounds ? kWaveRounds : per_wave;
    const uint64_t chunk = 64ull * rounds;
    unsigned long long carry = 0;
    for (uint64_t b = 0; b < nh; b += 1024 * PER) {
        const uint64_t k0 = b + (uint64_t)threadIdx.x * PER;
        unsigned long long v[PER], sum = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            v[q] = k0 + q < nh ? (unsigned long long)hits[k0 + q].count : 0ull;
            sum += v[q];
        }
        const unsigned long long incl = wave_incl_scan(sum);
        if (lane == 63) s_w[w] = incl;
        __syncthreads();
        unsigned long long at = carry + incl - sum, tot = 0;
        for (int q = 0; q < 16; ++q) {
            if (q < w) at += s_w[q];
            tot += s_w[q];
        }
        carry += tot;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (k0 + q < nh) {
                prefix[k0 + q] = at;
                for (uint64_t ch = (at + chunk - 1) / chunk; ch * chunk < at + v[q]; ++ch)
                    first[ch] = (uint32_t)(k0 + q);
                at += v[q];
            }
        }
    }
    if (threadIdx.x == 0) {
        prefix[nh] = carry;
        bc[0] = nh;
        bc[1] = carry;
        bc[2] = (carry + chunk - 1) / chunk;
        bc[3] = flags;
        bc[4] = rounds;
    }
}

// One block: the batch's accepted (gx, gy) become (query id << 32 | indexed id) keys, sorted in
// LDS (bitonic), deduplicated and compacted in order, after the batch's counters: the result block.
// More than kGraphSortCap accepted pairs, or more than the accepted buffer held, sets a flag and
// outputs nothing.
__global__ __launch_bounds__(1024) void k_batch_dedupe(const uint64_t* __restrict__ acc,
                                                       const unsigned long long* __restrict__ counters,
                                                       uint64_t acc_cap,
                                                       const int32_t* __restrict__ xperm,
                                                       const int32_t* __restrict__ yperm,
                                                       const unsigned long long* __restrict__ bc,
                                                       unsigned long long* __restrict__ result)
{
    __shared__ uint64_t s_k[kGraphSortCap];
    __shared__ uint32_t s_w[16];
    uint64_t* out = (uint64_t*)(result + kBatchResultHead);
    const uint64_t m = counters[3];
    const bool over = m > acc_cap || m > (uint64_t)kGraphSortCap;
    if (threadIdx.x < 8) {
        result[threadIdx.x] = counters[threadIdx.x];
    } else if (threadIdx.x < 12) {
        const int k = (int)threadIdx.x - 8;
        result[threadIdx.x] = bc[k] | (k == 3 && over ? (m > acc_cap ? 4ull : 0ull) | 8ull : 0ull);
    }
    if (over) {
        if (threadIdx.x == 0) result[12] = 0;
        return;
    }
    uint32_t N = 64;
    while (N < (uint32_t)m) N <<= 1;
    for (uint32_t k = threadIdx.x; k < N; k += 1024) {
        uint64_t key = ~0ull;
        if (k < (uint32_t)m) {
            const uint64_t v = acc[k];
            const uint32_t a = (uint32_t)xperm[v >> 32];
            const uint32_t b = (uint32_t)yperm[v & 0xffffffffu];
            key = ((uint64_t)a << 32) | b;
        }
        s_k[k] = key;
    }
    __syncthreads();
    block_bitonic_sort(s_k, N, 1024u);
    uint32_t carry = 0;
    for (uint32_t base = 0; base < (uint32_t)m; base += 1024) {
        const uint32_t k = base + threadIdx.x;
        const bool head = k < (uint32_t)m && (k == 0 || s_k[k] != s_k[k - 1]);
        uint32_t tot;
        const uint32_t at = carry + block_rank_1024(head, s_w, &tot);
        if (head) out[at] = s_k[k];
        carry += tot;
    }
    if (threadIdx.x == 0) result[12] = carry;
}

template <int W>
static void graph_verify_short(const GraphBatch& G, hipStream_t s)
{
    verify_batched_w<W>(G.verify, G.first, 0, G.verify_grid, s);
    if (G.y_count) {
        const ProbeParams& P = G.probe;
        const unsigned grid = G.y_count < 65536 ? G.y_count : 65536;
        hipLaunchKernelGGL((k_short<W>), dim3(grid), dim3(kBlock), 0, s, P.x_arena, P.x_slen,
                           P.x_lenstart, P.x_gbase, kLenMax, G.y_arena, G.y_slen, G.y_lenstart,
                           G.y_gbase, G.y_first, G.y_count, P.tau, 0, P.q_tau, G.verify.out,
                           G.verify.out_cap, 0, G.verify.counters);
    }
}

hipError_t launch_graph_probe(const GraphBatch& G, hipStream_t s)
{
    if (!G.probe.nx_dev || !G.verify.dev_counts || G.probe_grid < 1 || G.verify_grid < 1)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_probe, dim3(G.probe_grid), dim3(kBlock), 0, s, G.probe,
                       make_div(G.probe.tau + 1));
    return hipGetLastError();
}

hipError_t launch_graph_verify(const GraphBatch& G, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_prefix, dim3(1), dim3(1024), 0, s, G.probe.hits, G.probe.counters,
                       G.probe.hit_cap, const_cast<unsigned long long*>(G.verify.prefix), G.bcounts,
                       G.first, G.cand_cap);
    const int w = G.verify.tau + 1;
    if (w <= 9) graph_verify_short<9>(G, s);
    else if (w <= 17) graph_verify_short<17>(G, s);
    else if (w <= 33) graph_verify_short<33>(G, s);
    else graph_verify_short<64>(G, s);
    hipLaunchKernelGGL(k_batch_dedupe, dim3(1), dim3(1024), 0, s, G.verify.out,
                       G.verify.counters, G.verify.out_cap, G.xperm, G.yperm, G.bcounts, G.result);
    return hipGetLastError();
}

hipError_t launch_pairs_to_keys(const uint64_t* acc, uint64_t m, const int32_t* xperm,
                                const int32_t* yperm, int self, int bbits, uint64_t* keys,
                                hipStream_t s)
{
    if (m == 0) return hipSuccess;
    hipLaunchKernelGGL(k_pairs_to_keys, dim3(blocks_for(m)), dim3(kBlock), 0, s, acc, m, xperm,
                       yperm, self, bbits, keys);
    return hipGetLastError();
}

// Streamed self-joins: a window's result pairs (window-local ids) as global sort keys
// ids[a] << bbits | ids[b].  With min_len > 0 a pair of two strings shorter than min_len (both
// in the window's halo, found again by the window that owns them) becomes the sentinel, all
// ones in 2 * bbits bits, which no pair (a < b) reaches and which sorts after every pair; the
// sentinels are counted.
__global__ __launch_bounds__(kBlock) void k_window_keys(const int32_t* __restrict__ a,
                                                       const int32_t* __restrict__ b, uint64_t m,
                                                       const int32_t* __restrict__ ids,
                                                       const int32_t* __restrict__ offs,
                                                       int min_len, int bbits,
                                                       uint64_t* __restrict__ keys,
                                                       unsigned long long* __restrict__ dropped)
{
    const uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    bool drop = false;
    if (k < m) {
        const int32_t la = a[k], lb = b[k];
        if (min_len > 0) {
            const int na = offs[la + 1] - offs[la], nb = offs[lb + 1] - offs[lb];
            drop = (na > nb ? na : nb) < min_len;
        }
        keys[k] = drop ? ((2 * bbits >= 64) ? ~0ull : (1ull << (2 * bbits)) - 1ull)
                       : ((uint64_t)(uint32_t)ids[la] << bbits) | (uint64_t)(uint32_t)ids[lb];
    }
    const uint64_t dm = __ballot(drop);
    if ((threadIdx.x & 63) == 0 && dm) atomicAdd(dropped, (unsigned long long)__popcll(dm));
}

__global__ __launch_bounds__(kBlock) void k_split_keys(const uint64_t* __restrict__ keys,
                                                      uint64_t m, int bbits,
                                                      int32_t* __restrict__ a,
                                                      int32_t* __restrict__ b)
{
    const uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k < m) {
        const uint64_t v = keys[k];
        a[k] = (int32_t)(v >> bbits);
        b[k] = (int32_t)(v & ((1ull << bbits) - 1));
    }
}

hipError_t launch_window_keys(const int32_t* a, const int32_t* b, uint64_t m, const int32_t* ids,
                              const int32_t* offs, int min_len, int bbits, uint64_t* keys,
                              unsigned long long* dropped, hipStream_t s)
{
    if (m == 0) return hipSuccess;
    if (bbits < 1 || bbits > 31) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_window_keys, dim3(blocks_for(m)), dim3(kBlock), 0, s, a, b, m, ids, offs,
                       min_len, bbits, keys, dropped);
    return hipGetLastError();
}

hipError_t launch_split_keys(const uint64_t* keys, uint64_t m, int bbits, int32_t* a, int32_t* b,
                             hipStream_t s)
{
    if (m == 0) return hipSuccess;
    if (bbits < 1 || bbits > 31) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_split_keys, dim3(blocks_for(m)), dim3(kBlock), 0, s, keys, m, bbits, a, b);
    return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_fill_words(uint32_t* __restrict__ p, uint64_t n,
                                                       uint32_t v)
{
    for (uint64_t k = (uint64_t)blockIdx.x * kBlock + threadIdx.x; k < n;
         k += (uint64_t)gridDim.x * kBlock)
        p[k] = v;
}

hipError_t launch_fill_words(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const unsigned grid = (unsigned)std::min<uint64_t>(blocks_for(n), 4096);
    hipLaunchKernelGGL(k_fill_words, dim3(grid), dim3(kBlock), 0, s, p, n, v);
    return hipGetLastError();
}

// Checksum of a device string set: offsets[0 .. n] and bytes[0 .. min(offsets[n], cap)) as 8-byte words
// (the last padded with zeros), each element mixed (SplitMix64's finaliser; words before and after
// their index is added) and summed.  A plan compares it with the value taken when it was made; cap
// (the bytes allocation measured then) bounds the reads whatever offsets[n] holds now.  10^6 short
// strings: byte by byte, with an atomic a wave, 114 us, 16 bytes at a time and an atomic a block 19.
__global__ __launch_bounds__(kBlock) void k_set_checksum(const int32_t* __restrict__ offs, int64_t n,
                                                         const uint8_t* __restrict__ bytes,
                                                         int64_t cap,
                                                         unsigned long long* __restrict__ sum)
{
    const int64_t last = offs[n];
    const int64_t total = bytes ? (last < 0 ? 0 : (last < cap ? last : cap)) : 0;
    uint64_t acc = 0;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k <= n; k += stride)
        acc += mix64((uint64_t)(uint32_t)offs[k] ^ ((uint64_t)k << 32) ^ 0x243F6A8885A308D3ull);
    auto word = [&](uint64_t v, uint64_t index) {
        acc += mix64(mix64(v ^ 0x13198A2E03707344ull) + index * 0x9E3779B97F4A7C15ull);
    };
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; 16 * k < total; k += stride) {
        uint64_t v[2] = {0, 0};
        if (16 * k + 16 <= total) {
            const Unaligned16 c = *reinterpret_cast<const Unaligned16*>(bytes + 16 * k);
            v[0] = (uint64_t)c.w[1] << 32 | c.w[0];
            v[1] = (uint64_t)c.w[3] << 32 | c.w[2];
        } else {
            for (int64_t q = 16 * k; q < total; ++q)
                v[(q >> 3) & 1] |= (uint64_t)bytes[q] << (8 * (q & 7));
        }
        word(v[0], (uint64_t)(2 * k));
        word(v[1], (uint64_t)(2 * k + 1));
    }
    block_add(sum, acc);
}

hipError_t launch_set_checksum(const int32_t* offs, int64_t n, const uint8_t* bytes, int64_t cap,
                               unsigned long long* sum, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_words, dim3(1), dim3(kBlock), 0, s, (uint32_t*)sum, (uint64_t)2, 0u);
    const unsigned grid = (unsigned)std::max<uint64_t>(
        1, std::min<uint64_t>(blocks_for((uint64_t)n + 1), 1024));
    hipLaunchKernelGGL(k_set_checksum, dim3(grid), dim3(kBlock), 0, s, offs, n, bytes, cap, sum);
    return hipGetLastError();
}

hipError_t launch_gather_i32(const int32_t* in, const int32_t* perm, int64_t n, int32_t* out,
                             hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_i32, dim3(blocks_for(n)), dim3(kBlock), 0, s, in, perm, n, out);
    return hipGetLastError();
}

}  // namespace pj

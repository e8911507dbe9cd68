// pj_automaton.hip -- list-segment verification with the parts' DPs as table reads (thresholds up
// to 4, indexed strings of up to 47 bytes).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pj_automaton.h"
#include "pj_device_common.h"
#include "pj_internal.h"

namespace pj {

template <int TMAX>
__device__ const AutoTable<TMAX> d_auto{};

constexpr int kAutoBlock = 1024, kAutoWaves = kAutoBlock / 64;
// Position masks: bit q + kFirstBit of character c's mask says that the probe's character q is c.
// The low word of an entry holds bits 0 .. 31 and the high one bits kHighBit .. kHighBit + 31, so
// that the bits of four rows are in one word: q <= 50 for strings of up to kAutoMaxLen + 4 bytes.
constexpr int kFirstBit = kAutoTau + 1, kHighBit = 24;
static_assert(kHighBit - 1 + 3 + kAutoWidth <= 31, "four rows' bits in the low word");
static_assert(kAutoMaxLen + kAutoTau - 1 + kFirstBit <= kHighBit + 31, "the last character's bit");

template <typename T>
using Lds = __attribute__((address_space(3))) T*;

struct __attribute__((packed)) Chars8 {
    uint32_t w[2];
};
struct __attribute__((packed)) Chars4 {
    uint32_t w;
};

// The same value, which the compiler takes for any other: uniform loads through such a pointer stay
// where they are written, in place of dozens of values held (and spilled) across all loops.
template <typename T>
__device__ inline const T* here(const T* p)
{
    asm("" : "+s"(p));
    return p;
}

// One part of a hit's candidates, the same for every lane: y[yo, yo + yl) against the probe's
// characters [xo, xo + xl), threshold t.
struct Part {
    int yo, yl, nr;             // nr: rows of the band
    int sh;                     // bit below the first row's (column's) window in the masks
    int a, mb, fb;
    int slack;                  // t - delta; the part passes with an entry's distance up to this
    bool columns;               // steps over the band's columns: |y part| > |x part|
    uint32_t init, dead;
};

template <int TMAX>
__device__ inline Part make_part(int xo, int xl, int yo, int yl, int t)
{
    Part P;
    P.columns = yl > xl;
    const int delta = P.columns ? yl - xl : xl - yl;
    P.yo = yo;
    P.yl = yl;
    P.nr = P.columns ? xl : yl;
    P.slack = t - delta;
    // (no table for delta > t: the part fails, and the first one is read for nothing)
    const int at = P.slack < 0 ? 0 : AutoTable<TMAX>::index(t, delta, P.columns ? 1 : 0);
    const uint32_t* gp = reinterpret_cast<const uint32_t*>(d_auto<TMAX>.geom + at);
    // init[0 .. 5] | dead | a, fields
    const int p0 = xl < kAutoWidth ? xl : kAutoWidth;
    const uint32_t iw = uniform_load(gp + (p0 >> 1)), gw = uniform_load(gp + 3);
    P.init = (p0 & 1) ? iw >> 16 : iw & 0xffffu;
    P.dead = gw & 0xffffu;
    P.a = (int)((gw >> 16) & 255u);
    P.mb = (int)((gw >> 24) & 15u);
    P.fb = (int)(gw >> 28);
    P.sh = xo + kFirstBit - 1 - P.a;
    return P;
}

// A lane's candidate (y: its part's characters): row (or column) r + 1 takes the masks' bits for the
// positions r + 1 - a .. r + 1 + b of the part as the equal characters, puts them into the entry's
// low bits and reads the next entry.  Characters around the part and behind it are real ones of the
// strings or the bytes after them: a cell left of the first position is never reached, and one past
// the last changes no row that counts.  passes: rows of the band with a value up to t (a prefix of
// the rows).  Returns the last entry, dead if the wave stopped before the last row.
template <bool COLUMNS>
__device__ inline uint32_t run_part(const Part& P, const uint8_t* y, uint32_t pos, uint32_t next,
                                    bool act, int& passes)
{
    const uint32_t mask = ((1u << P.mb) - 1u) << 1;
    uint32_t entry = act ? P.init : P.dead;
    int count = 0;
    if (COLUMNS) count = act && P.init != P.dead ? (int)((P.init & mask) >> (1 + P.fb)) - P.a : 0;
    uint64_t live = 0;
    auto row = [&](uint32_t word, int s, int r) {
        const uint32_t m = word >> s;
        entry = *(Lds<const uint16_t>)(uintptr_t)(next + (entry ^ ((entry ^ m) & mask)));
        asm("" : "+v"(entry));           // (a 32-bit value: not masked to 16 bits again)
        const bool alive = entry != P.dead;
        live = __builtin_amdgcn_ballot_w64(alive);
        if (COLUMNS) {
            const int top = (int)((entry & mask) >> (1 + P.fb)) + (r + 1 - P.a);
            count = max(count, alive ? top : 0);
        } else count += alive ? 1 : 0;
    };
    // Straight-line code, left at the first pair of rows after which no lane is live (the empty
    // statements keep the compiler from joining the tests into one of many scalar operations)
    int yl = P.yl, sh = P.sh;
    asm volatile("" : "+s"(yl), "+s"(sh));     // what follows from them is computed where it is used
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (yl <= 8 * q) goto done;
        const Chars8 v = *reinterpret_cast<const Chars8*>(y + 8 * q);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int r = 8 * q + 4 * g;
            // the masks of four rows first: they do not depend on the state
            const bool high = sh + r >= kHighBit;
            const uint32_t base = pos + (high ? 4u : 0u);
            const int s = sh + r - (high ? kHighBit : 0);
            uint32_t word[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                word[u] = *(Lds<const uint32_t>)(uintptr_t)(
                    base + 8u * ((v.w[g] >> (8 * u)) & 255u));
            if (yl >= r + 4) {
                row(word[0], s, r);
                row(word[1], s + 1, r + 1);
                if (live == 0) goto done;
                row(word[2], s + 2, r + 2);
                row(word[3], s + 3, r + 3);
                if (live == 0) goto done;
                asm volatile("");
                if (yl == r + 4) goto done;
            } else {
                row(word[0], s, r);
                if (yl == r + 1) goto done;
                row(word[1], s + 1, r + 1);
                if (yl == r + 2) goto done;
                asm volatile("");
                if (live == 0) goto done;
                row(word[2], s + 2, r + 2);
                goto done;
            }
        }
    }
    // (parts of more than 16 characters that are still live: one row at a time)
    for (int r = 16; r < yl && live != 0; ++r) {
        const bool high = sh + r >= kHighBit;
        const uint32_t word =
            *(Lds<const uint32_t>)(uintptr_t)(pos + (high ? 4u : 0u) + 8u * (uint32_t)y[r]);
        row(word, sh + r - (high ? kHighBit : 0), r);
    }
done:
    passes = count;
    return entry;
}

// The list kernel of k_verify_segs (segments of 64 members of a probed list, chunks of segments,
// left parts first, right parts of the survivors from a queue) with run_part in place of the banded
// DP.  That DP took 171 VALU and 167 scalar operations per 64 candidates, each unit 85 % busy.  A
// row is 6 VALU operations and two LDS reads here in place of some 27 at t = 4, and no string is
// staged in LDS; what is left is set-up by hit and control, 87 and 94 operations.  A block holds
// the tables once (3.8 KB up to t = 3, 22.3 KB with t = 4) for 16 waves, so that two blocks fill a
// CU.  10^6 short strings at tau = 4 (9.2 x 10^9 candidates): 46.3 -> 27.1 ms; 4x10^5 against 5x10^4
// at tau = 3: 336 -> 285 us.
template <int TMAX>
__global__ __launch_bounds__(kAutoBlock)
__attribute__((amdgpu_waves_per_eu(8)))
void k_verify_auto(VerifyParams V_, Div div, const Hit* __restrict__ big,
                   const uint32_t* __restrict__ segp, uint64_t nseg,
                   const uint32_t* __restrict__ first, uint64_t nchunks, uint32_t seg_chunk,
                   unsigned long long* ticket)
{
    constexpr int kCap = 112;                              // pairs buffered per wave
    constexpr int kCells = kAutoMaxLen + 1;                // rows of a part: 0 .. kAutoMaxLen
    __shared__ __attribute__((aligned(64))) uint16_t s_next[AutoTable<TMAX>::kBytes / 2];
    __shared__ __attribute__((aligned(16))) uint64_t s_pos[kAutoWaves][256];
    __shared__ uint64_t s_acc[kAutoWaves][kCap];
    __shared__ uint32_t s_q[kAutoWaves][128];              // left-part survivors
    __shared__ uint16_t s_cells[kAutoWaves][2][kCells];    // band cells in rows 1..s of either part
    // the parameters, read where they are used
    const VerifyParams* VP =
        reinterpret_cast<const VerifyParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int k = threadIdx.x; k < AutoTable<TMAX>::kBytes / 16; k += kAutoBlock)
        reinterpret_cast<uint4*>(s_next)[k] =
            reinterpret_cast<const uint4*>(d_auto<TMAX>.next)[k];
    for (int k = lane; k < 256; k += 64) s_pos[w][k] = 0;
    __syncthreads();
    WaveAppender<uint64_t, kCap> acc{s_acc[w], 0};
    const Lds<uint32_t> sq = (Lds<uint32_t>)s_q[w];
    const Lds<uint16_t> cells0 = (Lds<uint16_t>)s_cells[w][0];
    const Lds<uint16_t> cells1 = (Lds<uint16_t>)s_cells[w][1];
    const uint32_t next = (uint32_t)(uintptr_t)(Lds<const uint8_t>)s_next;
    const uint32_t pos = (uint32_t)(uintptr_t)(Lds<const uint8_t>)s_pos[w];
    const uint64_t wave = (uint64_t)blockIdx.x * kAutoWaves + (uint32_t)w;
    const uint64_t nwaves = (uint64_t)gridDim.x * kAutoWaves;
    auto lds_order = []() {        // a wave's LDS requests complete in order; so for the compiler too
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    uint64_t my_cells = 0, my_miss = 0;
    int n_old = 0;                                         // the masks' string: its length and
    uint32_t c_old = 0;                                    // this lane's character
    uint64_t ch = wave;
    while (ch < nchunks) {
        uint64_t sg_i = ch * seg_chunk;
        const uint64_t sg_end = (sg_i + seg_chunk < nseg) ? sg_i + seg_chunk : nseg;
        uint32_t h = uniform_load(first + ch);
        uint32_t sidx = (uint32_t)(sg_i - uniform_load(segp + h));
        uint32_t left_in_chunk = (uint32_t)(sg_end - sg_i);
        uint32_t cells = 0, miss = 0;          // of the chunk's candidates
        while (left_in_chunk > 0) {
            // everything about the hit is wave-uniform: probe string, slot, both parts
            const VerifyParams* V = here(VP);
            const uint32_t* hw = reinterpret_cast<const uint32_t*>(big + h);
            const uint32_t gx = uniform_load(hw), start = uniform_load(hw + 1);
            const uint32_t count = uniform_load(hw + 2), meta = uniform_load(hw + 3);
            int tau = uniform_load(&V->tau);
            const uint32_t* vals = uniform_load(&V->vals);
            Div dv = div;
            const int32_t* q_tau = uniform_load(&V->q_tau);
            if (q_tau) {
                tau = uniform_load(q_tau + gx);
                const IndexRef* rf = uniform_load(&V->refs) + tau;
                vals = uniform_load(&rf->vals);
                dv.d = (uint32_t)(tau + 1);
                dv.m = uniform_load(&rf->div_m);
            }
            const int p = (int)(meta & 2047u) + 1;
            const int i = (int)((meta >> 11) & 63u) + 1;
            const int l = (int)(meta >> 17);
            const int n = __builtin_amdgcn_readfirstlane((int)uniform_load(&V->x_slen)[gx]);
            const uint8_t* x = uniform_load(&V->x_arena) + uniform_load(uniform_load(&V->x_gbase) + n) +
                               (int64_t)(gx - (uint32_t)uniform_load(uniform_load(&V->x_lenstart) + n)) *
                                   stride_of(n);
            const Seg sgm = partition_seg(l, i, tau, dv);
            // position masks of x, one character a lane (n <= 51): the old string's out, the new
            // one's in
            const uint32_t c_new = lane < n ? x[lane] : 0u;
            if (lane < n_old) s_pos[w][c_old] = 0;
            lds_order();
            if (lane < n) {
                const int bit = lane + kFirstBit;
                const uint32_t lo = bit < 32 ? 1u << bit : 0u;
                const uint32_t hi = bit >= kHighBit ? 1u << (bit - kHighBit) : 0u;
                atomicOr((unsigned long long*)&s_pos[w][c_new], (uint64_t)hi << 32 | lo);
            }
            n_old = n;
            c_old = c_new;
            // left parts: x[1, p-1] vs y[1, p_i-1] with t = i-1; right parts after the segment
            // with t = tau+1-i (Algorithm 3)
            const int ry = sgm.p - 1 + sgm.len, rx = p - 1 + sgm.len;
            const Part L = make_part<TMAX>(0, p - 1, 0, sgm.p - 1, i - 1);
            const Part R = make_part<TMAX>(rx, n - rx, ry, l - ry, tau + 1 - i);
            // cells in the first rows of either part's band (Lemma 4)
            auto cells_of = [&](int xl, int yl, int t, Lds<uint16_t> out) {
                const int nr = min(xl, yl), nc = max(xl, yl), delta = nc - nr;
                if (delta <= t && lane <= nr)
                    out[lane] = (uint16_t)band_cells(lane, nc, (t - delta) >> 1, (t + delta) >> 1);
            };
            cells_of(p - 1, sgm.p - 1, i - 1, cells0);
            cells_of(n - rx, l - ry, tau + 1 - i, cells1);
            lds_order();
            const uint32_t hsegs = (count + 63u) / 64u;
            const uint32_t s_stop = hsegs - sidx < left_in_chunk ? hsegs : sidx + left_in_chunk;
            left_in_chunk -= s_stop - sidx;
            // with inline copies, entry e's string is at ystr + e * stride; else the string of
            // sorted position g at ystr + g * stride
            const uint32_t stride = (uint32_t)stride_of(l);
            const uint8_t* ystr = uniform_load(&V->y_inl);
            const bool inl = ystr != nullptr;
            if (inl) ystr += uniform_load(uniform_load(&V->y_inl_base) + l);
            else
                ystr = uniform_load(&V->y_arena) + uniform_load(uniform_load(&V->y_gbase) + l) -
                       (int64_t)uniform_load(uniform_load(&V->y_lenstart) + l) * stride;
            const int seg_bytes = sgm.len > uniform_load(&V->exact_len) ? sgm.len : 0;
            const uint64_t pair_x = (uint64_t)gx << 32;

            // a step of 64 candidates through a part: whether each passes
            auto step = [&](const Part& P, const uint8_t* y, Lds<uint16_t> ct, bool ok) -> bool {
                if (P.slack < 0) return false;
                int passes;
                const uint32_t entry =
                    P.columns ? run_part<true>(P, y + P.yo, pos, next, ok, passes)
                              : run_part<false>(P, y + P.yo, pos, next, ok, passes);
                // rows evaluated: those that passed and the first that did not
                const uint32_t rows = (uint32_t)min(passes + 1, P.nr);
                const uint32_t cc = ct[rows];
                cells += ok ? cc : 0u;
                return ok && (int)((entry >> 1) & ((1u << P.fb) - 1u)) <= P.slack;
            };
            // the hit's members [64 * sidx, ..): every lane takes a valid one (those past the end
            // repeat the last); string positions are needed early without inline copies only
            auto member = [&](uint32_t& src, bool& ok) -> const uint8_t* {
                const uint32_t m = sidx * 64u + (uint32_t)lane;
                ok = m < count;
                src = start + min(m, count - 1u);
                if (!inl) src = vals[src];
                const uint8_t* y = ystr + (uint64_t)src * stride;
                if (seg_bytes) {
                    // hashed key: the segment's bytes, four at a time
                    bool same = true;
                    for (int q = 0; q < seg_bytes; q += 4) {
                        const uint32_t yw = reinterpret_cast<const Chars4*>(y + sgm.p - 1 + q)->w;
                        uint32_t xw = 0;
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            xw |= (uint32_t)__builtin_amdgcn_readlane((int)c_new,
                                                                      (p - 1 + q + u) & 63) << (8 * u);
                        const int rest = seg_bytes - q;
                        const uint32_t in = rest >= 4 ? ~0u : (1u << (8 * rest)) - 1u;
                        same &= ((xw ^ yw) & in) == 0;
                    }
                    miss += (ok && !same) ? 1u : 0u;
                    ok = ok && same;
                }
                return y;
            };
            auto emit = [&](uint32_t src, bool ok) {
                if (__builtin_amdgcn_ballot_w64(ok) == 0) return;
                const uint32_t gy = inl ? vals[src] : src;
                const VerifyParams* VO = here(VP);
                acc.push(ok, pair_x | gy, uniform_load(&VO->out), uniform_load(&VO->out_cap),
                         uniform_load(&VO->counters) + 3);
            };
            // a part of two empty strings passes with no cells: the other part then runs on the
            // members directly
            const bool left_trivial = (p == 1) && (sgm.p == 1);
            const bool right_trivial = (rx == n) && (ry == l);
            if (left_trivial || right_trivial) {
                const Lds<uint16_t> ct = left_trivial ? cells1 : cells0;
                Part P = R;
                if (!left_trivial) P = L;
                for (; sidx < s_stop; ++sidx) {
                    uint32_t src;
                    bool ok;
                    const uint8_t* y = member(src, ok);
                    emit(src, step(P, y, ct, ok));
                }
            } else {
                uint32_t qn = 0;               // queued survivors: index entries (or positions)
                for (;;) {
                    if (sidx < s_stop) {
                        uint32_t src;
                        bool ok;
                        const uint8_t* y = member(src, ok);
                        ok = step(L, y, cells0, ok);
                        ++sidx;
                        const uint64_t surv = __builtin_amdgcn_ballot_w64(ok);
                        if (surv != 0) {
                            // appended in lane order; qn < 64, so the last word is never an entry
                            // and takes the other lanes' writes
                            const uint32_t at =
                                qn + __builtin_amdgcn_mbcnt_hi(
                                         (uint32_t)(surv >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)surv, 0u));
                            sq[ok ? at : 127u] = src;
                            qn += (uint32_t)__builtin_popcountll(surv);
                        }
                        if (qn < 64u) continue;
                    }
                    if (qn == 0) break;
                    lds_order();
                    const uint32_t k = min(qn, 64u);
                    const bool ok = (uint32_t)lane < k;
                    const uint32_t src = sq[ok ? lane : 0];
                    // the rest of the queue to its front, all reads before the writes
                    const uint32_t mv = sq[64 + lane];
                    lds_order();
                    sq[lane] = mv;
                    qn -= k;
                    emit(src, step(R, ystr + (uint64_t)src * stride, cells1, ok));
                }
            }
            ++h;
            sidx = 0;
        }
        my_cells += cells;
        my_miss += miss;
        if (!ticket) break;                        // a chunk for every wave
        unsigned long long t = 0;
        if (lane == 0) t = atomicAdd(ticket, 1ull);
        ch = nwaves + ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)t) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(t >> 32)) << 32);
    }
    block_flush<kAutoWaves>(acc, V_.out, V_.out_cap, &V_.counters[3]);
    unsigned long long* line = stat_line(V_.counters, V_.shards);
    block_add<kAutoWaves>(&line[7], my_cells);
    block_add<kAutoWaves>(&line[5], my_miss);
}

hipError_t launch_verify_auto(const VerifyParams& V, const Hit* big, const uint32_t* segp,
                              uint64_t nseg, const uint32_t* first, uint64_t nchunks,
                              uint32_t chunk, uint64_t waves, unsigned long long* ticket,
                              hipStream_t s)
{
    if (V.tau > kAutoTau || V.y_maxlen > kAutoMaxLen) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((waves + kAutoWaves - 1) / kAutoWaves)), block(kAutoBlock);
    if (V.tau <= 3)
        hipLaunchKernelGGL((k_verify_auto<3>), grid, block, 0, s, V, make_div(V.tau + 1), big, segp,
                           nseg, first, nchunks, chunk, ticket);
    else
        hipLaunchKernelGGL((k_verify_auto<4>), grid, block, 0, s, V, make_div(V.tau + 1), big, segp,
                           nseg, first, nchunks, chunk, ticket);
    return hipGetLastError();
}

}  // namespace pj

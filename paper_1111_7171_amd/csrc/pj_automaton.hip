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

// One part of a hit's candidates, the same for every lane: |y part| yl against the probe's characters
// from xo on, threshold t.  Two words, set up by a lane (pack_part) and taken apart by the wave.
//   entries: init | dead << 16
//   shape: yl 0..5 | nr (rows of the band) 6..11 | sh (the bit below the first row's or column's
//          window in the masks) 12..17 | t - delta 18..20 | delta > t 21 | steps over the band's
//          columns (|y part| > |x part|) 22 | mb 23..25 | fb 26..27 | a 28..30
struct PackedPart {
    uint32_t entries;           // init | dead << 16
    uint32_t shape;
    uint32_t cells;             // of the part's row in the table of cells
};

template <int TMAX>
__device__ inline PackedPart pack_part(int xo, int xl, int yl, int t)
{
    PackedPart R;
    const bool columns = yl > xl;
    const int delta = columns ? yl - xl : xl - yl, nr = columns ? xl : yl;
    const bool fails = delta > t;
    // (no table for delta > t: the first one is read for nothing)
    const int at = fails ? 0 : AutoTable<TMAX>::index(t, delta, columns ? 1 : 0);
    const uint4 g = *reinterpret_cast<const uint4*>(d_auto<TMAX>.geom + at);
    // init[0 .. 5] | dead | a, fields: row 0 with xl positions, of which kAutoWidth at most matter
    const int p0 = xl < kAutoWidth ? xl : kAutoWidth;
    const uint32_t iw = p0 < 2 ? g.x : p0 < 4 ? g.y : g.z;
    const uint32_t a = (g.w >> 16) & 255u, mb = (g.w >> 24) & 15u, fb = g.w >> 28;
    R.entries = ((p0 & 1) ? iw >> 16 : iw & 0xffffu) | g.w << 16;
    const uint32_t sh = (uint32_t)(xo + kFirstBit - 1) - a;
    R.shape = (uint32_t)yl | (uint32_t)nr << 6 | sh << 12 | (uint32_t)((t - delta) & 7) << 18 |
              (fails ? 1u << 21 : 0u) | (columns ? 1u << 22 : 0u) | mb << 23 | fb << 26 | a << 28;
    R.cells = (uint32_t)(((at >> 1) * AutoTable<TMAX>::kCellRows + nr) * AutoTable<TMAX>::kCellRows);
    return R;
}

struct Part {
    int yl, nr, sh, slack, a, fb;
    bool fails, columns;
    uint32_t mask, init, dead;  // mask: the characters' bits in an entry
};

__device__ inline Part unpack_part(uint32_t entries, uint32_t shape)
{
    Part P;
    P.yl = (int)(shape & 63u);
    P.nr = (int)(shape >> 6 & 63u);
    P.sh = (int)(shape >> 12 & 63u);
    P.slack = (int)(shape >> 18 & 7u);
    P.fails = shape >> 21 & 1u;
    P.columns = shape >> 22 & 1u;
    P.mask = ((1u << (shape >> 23 & 7u)) - 1u) << 1;
    P.fb = (int)(shape >> 26 & 3u);
    P.a = (int)(shape >> 28);
    P.init = entries & 0xffffu;
    P.dead = entries >> 16;
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
                                    uint64_t act, int& passes)
{
    const uint32_t mask = P.mask, dead = P.dead;
    const bool in = __builtin_amdgcn_inverse_ballot_w64(act);
    uint32_t entry = in ? P.init : dead;
    int count = 0;
    if (COLUMNS && P.init != dead) count = in ? (int)((P.init & mask) >> (1 + P.fb)) - P.a : 0;
    uint64_t live = 0;
    auto row = [&](uint32_t word, int s, int r) {
        const uint32_t m = word >> s;
        entry = *(Lds<const uint16_t>)(uintptr_t)(next + (entry ^ ((entry ^ m) & mask)));
        asm("" : "+v"(entry));           // (a 32-bit value: not masked to 16 bits again)
        const bool alive = entry != dead;
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
// staged in LDS.  What is left is control and set-up by hit, about 80 operations of either kind per 64
// candidates (each unit 75 % busy), and waiting (four waves of eight): a hit's set-up, 250 scalar operations when every wave did
// it for itself, is done for 64 hits at once, a lane each.  A block holds the tables once (3.8 KB up
// to t = 3, 22.3 KB with t = 4) for 16 waves, so that two blocks fill a CU.  10^6 short strings at
// tau = 4 (9.2 x 10^9 candidates): banded DP 46.3 ms, tables 27.1, set-up by lanes 24.6.
struct AutoArgs {
    VerifyParams V;
    Div div;
    const Hit* big;
    const uint32_t* segp;
    const uint32_t* first;
    unsigned long long* ticket;
    uint64_t nseg, nchunks;
    uint32_t nbig, seg_chunk;
};

template <int TMAX>
__global__ __launch_bounds__(kAutoBlock)
__attribute__((amdgpu_waves_per_eu(8)))
void k_verify_auto(AutoArgs)
{
    constexpr int kCap = 136;                              // pairs buffered per wave
    __shared__ __attribute__((aligned(64))) uint16_t s_next[AutoTable<TMAX>::kBytes / 2];
    __shared__ __attribute__((aligned(16))) uint64_t s_pos[kAutoWaves][256];
    __shared__ uint64_t s_acc[kAutoWaves][kCap];
    __shared__ uint32_t s_q[kAutoWaves][128];              // left-part survivors
    // the parameters, read where they are used
    const AutoArgs* AP =
        reinterpret_cast<const AutoArgs*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int k = threadIdx.x; k < AutoTable<TMAX>::kBytes / 16; k += kAutoBlock)
        reinterpret_cast<uint4*>(s_next)[k] =
            reinterpret_cast<const uint4*>(d_auto<TMAX>.next)[k];
    for (int k = lane; k < 256; k += 64) s_pos[w][k] = 0;
    __syncthreads();
    WaveAppender<uint64_t, kCap> acc{s_acc[w], 0};
    const Lds<uint32_t> sq = (Lds<uint32_t>)s_q[w];
    const uint32_t next = (uint32_t)(uintptr_t)(Lds<const uint8_t>)s_next;
    const uint32_t pos = (uint32_t)(uintptr_t)(Lds<const uint8_t>)s_pos[w];
    const uint64_t wave = (uint64_t)blockIdx.x * kAutoWaves + (uint32_t)w;
    auto lds_order = []() {        // a wave's LDS requests complete in order; so for the compiler too
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    uint64_t my_cells = 0;
    int n_old = 0;                                         // the masks' string: its length and
    uint32_t c_old = 0;                                    // this lane's character
    uint32_t tried = 0;
    uint64_t ch = wave;
    while (ch < uniform_load(&here(AP)->nchunks)) {
        const AutoArgs* C = here(AP);
        const uint32_t seg_chunk = uniform_load(&C->seg_chunk);
        const uint64_t nseg = uniform_load(&C->nseg);
        const uint64_t sg_i = ch * seg_chunk;
        const uint64_t sg_end = (sg_i + seg_chunk < nseg) ? sg_i + seg_chunk : nseg;
        uint32_t h = uniform_load(uniform_load(&C->first) + ch);
        uint32_t sidx = (uint32_t)(sg_i - uniform_load(uniform_load(&C->segp) + h));
        uint32_t left_in_chunk = (uint32_t)(sg_end - sg_i);
        uint32_t cells = 0, miss = 0;          // of the chunk's candidates
        while (left_in_chunk > 0) {
            // Hits h .. h + 63, a lane each: what the wave needs of a hit comes from the lane's
            // registers then (13 reads in place of some 250 scalar operations and three loads one
            // after another a hit; lists have four segments on average where this matters most)
            const AutoArgs* H = here(AP);
            const VerifyParams* V = &H->V;
            const Hit* hp = uniform_load(&H->big) +
                            min(h + (uint32_t)lane, uniform_load(&H->nbig) - 1u);
            const uint4 hw = *reinterpret_cast<const uint4*>(hp);
            const uint32_t v_gx = hw.x, v_start = hw.y, v_count = hw.z, meta = hw.w;
            int tau = uniform_load(&V->tau);
            Div dv;
            dv.m = uniform_load(&H->div.m);
            dv.d = uniform_load(&H->div.d);
            const int32_t* q_tau = uniform_load(&V->q_tau);
            if (q_tau) {
                tau = q_tau[v_gx];
                const IndexRef* rf = uniform_load(&V->refs) + tau;
                dv.d = (uint32_t)(tau + 1);
                dv.m = rf->div_m;
            }
            const int p = (int)(meta & 2047u) + 1;
            const int i = (int)((meta >> 11) & 63u) + 1;
            const int l = (int)(meta >> 17);
            const int n = uniform_load(&V->x_slen)[v_gx];
            const uint64_t v_x = (uint64_t)(uniform_load(&V->x_gbase)[n] +
                                            (int64_t)(v_gx - (uint32_t)uniform_load(&V->x_lenstart)[n]) *
                                                stride_of(n));
            // with inline copies, entry e's string is at ybase + e * stride; else the string of
            // sorted position g at ybase + g * stride
            const uint8_t* yall = uniform_load(&V->y_inl);
            const bool inl = yall != nullptr;
            uint64_t v_y;
            if (inl) v_y = (uint64_t)uniform_load(&V->y_inl_base)[l];
            else {
                yall = uniform_load(&V->y_arena);
                v_y = (uint64_t)(uniform_load(&V->y_gbase)[l] -
                                 (int64_t)uniform_load(&V->y_lenstart)[l] * stride_of(l));
            }
            // left parts: x[1, p-1] vs y[1, p_i-1] with t = i-1; right parts after the segment
            // with t = tau+1-i (Algorithm 3)
            const Seg sgm = partition_seg(l, i, tau, dv);
            const int v_ry = sgm.p - 1 + sgm.len, v_rx = p - 1 + sgm.len;
            const PackedPart pl = pack_part<TMAX>(0, p - 1, sgm.p - 1, i - 1);
            const PackedPart pr = pack_part<TMAX>(v_rx, n - v_rx, l - v_ry, tau + 1 - i);
            // lengths and places, and whether a part is two empty strings
            const uint32_t v_where = (uint32_t)n | (uint32_t)l << 6 | (uint32_t)v_ry << 12 |
                                     (uint32_t)(sgm.p - 1) << 18 | (uint32_t)(p - 1) << 24 |
                                     (p == 1 && sgm.p == 1 ? 1u << 30 : 0u) |
                                     (v_rx == n && v_ry == l ? 1u << 31 : 0u);
            const uint32_t v_cells = pl.cells | pr.cells << 16;
            const uint8_t* xall = uniform_load(&V->x_arena);
            const int exact_len = uniform_load(&V->exact_len);
            auto at = [](uint32_t v, int k) {
                return (uint32_t)__builtin_amdgcn_readlane((int)v, k);
            };
            auto at64 = [&](uint64_t v, int k) {
                return (uint64_t)at((uint32_t)(v >> 32), k) << 32 | at((uint32_t)v, k);
            };
            // the probe strings' characters are loaded a hit ahead (64 of them lie in the arena)
            uint32_t c_next = (xall + at64(v_x, 0))[lane];
            for (int k = 0; k < 64 && left_in_chunk > 0; ++k) {
                const uint32_t where = at(v_where, k);
                const int nx = (int)(where & 63u);
                // position masks of x, one character a lane (n <= 51): the old string's out, the
                // new one's in
                const uint32_t c_new = c_next;
                if (k < 63) c_next = (xall + at64(v_x, k + 1))[lane];
                if (lane < n_old) s_pos[w][c_old] = 0;
                lds_order();
                if (lane < nx) {
                    const int bit = lane + kFirstBit;
                    const uint32_t lo = bit < 32 ? 1u << bit : 0u;
                    const uint32_t hi = bit >= kHighBit ? 1u << (bit - kHighBit) : 0u;
                    atomicOr((unsigned long long*)&s_pos[w][c_new], (uint64_t)hi << 32 | lo);
                }
                lds_order();
                n_old = nx;
                c_old = c_new;
                const uint32_t start = at(v_start, k), count = at(v_count, k);
                const int ly = (int)((where >> 6) & 63u), ry = (int)((where >> 12) & 63u);
                const int seg_len = ry - (int)((where >> 18) & 63u);
                const bool left_trivial = (where >> 30) & 1u, right_trivial = where >> 31;
                const uint32_t l_entries = at(pl.entries, k), l_shape = at(pl.shape, k);
                const uint32_t r_entries = at(pr.entries, k), r_shape = at(pr.shape, k);
                const uint32_t cell_rows = at(v_cells, k);
                const uint32_t stride = (uint32_t)stride_of(ly);
                const uint8_t* ystr = yall + at64(v_y, k);
                const int seg_bytes = seg_len > exact_len ? seg_len : 0;
                // the string positions of the hit's index
                auto positions = [&]() {
                    const VerifyParams* VO = &here(AP)->V;
                    const int32_t* qt = uniform_load(&VO->q_tau);
                    if (!qt) return uniform_load(&VO->vals);
                    int kk = k;
                    asm volatile("" : "+s"(kk));
                    return uniform_load(&(uniform_load(&VO->refs) +
                                          uniform_load(qt + at(v_gx, kk)))->vals);
                };
                const uint32_t hsegs = (count + 63u) / 64u;
                const uint32_t s_stop = hsegs - sidx < left_in_chunk ? hsegs : sidx + left_in_chunk;
                left_in_chunk -= s_stop - sidx;

                // a step of 64 candidates through a part: whether each passes
                auto step = [&](const Part& P, uint32_t ct, const uint8_t* y, uint64_t ok) {
                    if (P.fails) return (uint64_t)0;
                    int passes;
                    const uint32_t entry = P.columns ? run_part<true>(P, y, pos, next, ok, passes)
                                                     : run_part<false>(P, y, pos, next, ok, passes);
                    // rows evaluated: those that passed and the first that did not
                    const uint32_t cc = d_auto<TMAX>.cells[ct + (uint32_t)min(passes + 1, P.nr)];
                    cells += __builtin_amdgcn_inverse_ballot_w64(ok) ? cc : 0u;
                    return ok & __builtin_amdgcn_ballot_w64(
                                    (int)((entry >> 1) & ((1u << P.fb) - 1u)) <= P.slack);
                };
                // the hit's members [64 * sidx, ..): every lane takes a valid one (those past the
                // end repeat the last)
                auto member = [&](uint32_t& src, uint64_t& ok) -> const uint8_t* {
                    const uint32_t m = sidx * 64u + (uint32_t)lane;
                    ok = __builtin_amdgcn_ballot_w64(m < count);
                    src = start + min(m, count - 1u);
                    if (!inl) src = positions()[src];
                    const uint8_t* y = ystr + (uint64_t)src * stride;
                    if (seg_bytes) {
                        // hashed key: the segment's bytes, four at a time
                        uint32_t other = 0;
                        const int ys = (int)((where >> 18) & 63u), xs = (int)((where >> 24) & 63u);
                        for (int q = 0; q < seg_bytes; q += 4) {
                            const uint32_t yw = reinterpret_cast<const Chars4*>(y + ys + q)->w;
                            uint32_t xw = 0;
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                xw |= at(c_new, (xs + q + u) & 63) << (8 * u);
                            const int rest = seg_bytes - q;
                            const uint32_t in = rest >= 4 ? ~0u : (1u << (8 * rest)) - 1u;
                            other |= (xw ^ yw) & in;
                        }
                        const uint64_t same = __builtin_amdgcn_ballot_w64(other == 0);
                        miss += (uint32_t)__builtin_popcountll(ok & ~same);
                        ok &= same;
                    }
                    return y;
                };
                auto emit = [&](uint32_t src, uint64_t ok) {
                    if (ok == 0) return;
                    const uint32_t gy = inl ? positions()[src] : src;
                    const VerifyParams* VO = &here(AP)->V;
                    int kk = k;
                    asm volatile("" : "+s"(kk));
                    acc.push(__builtin_amdgcn_inverse_ballot_w64(ok),
                             (uint64_t)at(v_gx, kk) << 32 | gy, uniform_load(&VO->out), uniform_load(&VO->out_cap),
                             uniform_load(&VO->counters) + 3);
                };
                // a part of two empty strings passes with no cells: the other part then runs on
                // the members directly
                if (left_trivial || right_trivial) {
                    const uint32_t ct = left_trivial ? cell_rows >> 16 : cell_rows & 0xffffu;
                    const int yo = left_trivial ? ry : 0;
                    const Part P = unpack_part(left_trivial ? r_entries : l_entries,
                                               left_trivial ? r_shape : l_shape);
                    for (; sidx < s_stop; ++sidx) {
                        uint32_t src;
                        uint64_t ok;
                        const uint8_t* y = member(src, ok);
                        emit(src, step(P, ct, y + yo, ok));
                    }
                } else {
                    const Part L = unpack_part(l_entries, l_shape);
                    uint32_t qn = 0;           // queued survivors: index entries (or positions)
                    for (;;) {
                        if (sidx < s_stop) {
                            uint32_t src;
                            uint64_t ok;
                            const uint8_t* y = member(src, ok);
                            ok = step(L, cell_rows & 0xffffu, y, ok);
                            ++sidx;
                            if (ok != 0) {
                                // appended in lane order; qn < 64, so the last word is never an
                                // entry and takes the other lanes' writes
                                const uint32_t to =
                                    qn + __builtin_amdgcn_mbcnt_hi(
                                             (uint32_t)(ok >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)ok, 0u));
                                sq[__builtin_amdgcn_inverse_ballot_w64(ok) ? to : 127u] = src;
                                qn += (uint32_t)__builtin_popcountll(ok);
                            }
                            if (qn < 64u) continue;
                        }
                        if (qn == 0) break;
                        lds_order();
                        const uint32_t take = min(qn, 64u);
                        const bool in = (uint32_t)lane < take;
                        const uint32_t src = sq[in ? lane : 0];
                        // the rest of the queue to its front, all reads before the writes
                        const uint32_t mv = sq[64 + lane];
                        lds_order();
                        sq[lane] = mv;
                        qn -= take;
                        // (few steps a hit: the part is taken apart here, not held)
                        uint32_t entries = r_entries, shape = r_shape;
                        asm volatile("" : "+s"(entries), "+s"(shape));
                        emit(src, step(unpack_part(entries, shape), cell_rows >> 16,
                                       ystr + (uint64_t)src * stride + ry,
                                       __builtin_amdgcn_ballot_w64(in)));
                    }
                }
                ++h;
                sidx = 0;
            }
        }
        my_cells += cells;
        if (miss && lane == 0) {               // (hardly ever: keys that differ but hash alike)
            const VerifyParams* VM = &here(AP)->V;
            atomicAdd(&stat_line(uniform_load(&VM->counters), uniform_load(&VM->shards))[5],
                      (unsigned long long)miss);
        }
        const AutoArgs* D = here(AP);
        ch = next_chunk(uniform_load(&D->ticket), tried, (uint64_t)gridDim.x * kAutoWaves,
                        uniform_load(&D->nchunks));
    }
    const VerifyParams* V = &here(AP)->V;
    unsigned long long* counters = uniform_load(&V->counters);
    block_flush<kAutoWaves>(acc, uniform_load(&V->out), uniform_load(&V->out_cap), &counters[3]);
    unsigned long long* line = stat_line(counters, uniform_load(&V->shards));
    block_add<kAutoWaves>(&line[7], my_cells);
}

hipError_t launch_verify_auto(const VerifyParams& V, const Hit* big, uint64_t nbig,
                              const uint32_t* segp, uint64_t nseg, const uint32_t* first, uint64_t nchunks,
                              uint32_t chunk, uint64_t waves, unsigned long long* ticket,
                              hipStream_t s)
{
    if (V.tau > kAutoTau || V.y_maxlen > kAutoMaxLen || nbig == 0) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((waves + kAutoWaves - 1) / kAutoWaves)), block(kAutoBlock);
    const AutoArgs args{V, make_div(V.tau + 1), big, segp, first, ticket, nseg, nchunks,
                        (uint32_t)nbig, chunk};
    if (V.tau <= 3) hipLaunchKernelGGL((k_verify_auto<3>), grid, block, 0, s, args);
    else hipLaunchKernelGGL((k_verify_auto<4>), grid, block, 0, s, args);
    return hipGetLastError();
}

}  // namespace pj

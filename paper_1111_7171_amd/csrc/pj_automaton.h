// pj_automaton.h -- the verification DP of a part as a finite automaton, for thresholds up to 4.
//
// A row of the band of Lemma 4 holds W = a + b + 1 <= t + 1 expected distances
// D(i, k) = M(i, k) + |b - k|, and row i + 1 depends on row i and on which of the W columns'
// characters equal the row's: W bits.  A value above t can never come back to t (D does not
// decrease along a step), so values are kept as min(D, t + 1), and few rows remain that can occur:
// 2 to 77 for t <= 4.  Numbering them turns a row of the DP into one table read, next[state][bits].
// (The construction of universal Levenshtein automata, Schulz and Mihov 2002, for this band and
// stop rule.)  The tables are computed here at compile time, from the recurrence itself.
//
// State entries are 16-bit byte offsets of the state's row of entries in the table.  Rows are
// aligned to their size, so an entry's low bits are free: the reader replaces them by the
// characters' bits (bit 0 stays clear), and until then they say what the state means:
//   bits 1 .. fb         min(D(i, b), t + 1) - delta, the distance if row i is the last
//   bits fb + 1 .. mb    largest band index with D <= t (0 if there is none)
// The band index runs over the positions of one string while the steps run over the other's
// characters; with A = a and B = b the steps are the rows of the band, with A = b and B = a its columns
// (the recurrence is symmetric in the two).  The last cell has band index B either way.
#pragma once

#include <stdint.h>

namespace pj {

constexpr int kAutoTau = 4;                      // largest threshold with a table
constexpr int kAutoWidth = kAutoTau + 1;

constexpr int auto_bits(int v) { return v == 0 ? 0 : 1 + auto_bits(v >> 1); }

// Geometry of part threshold t, length difference delta; steps over the band's columns or rows.
struct AutoShape {
    int t, delta, columns;
    constexpr int a() const { return columns ? (t + delta) >> 1 : (t - delta) >> 1; }
    constexpr int b() const { return columns ? (t - delta) >> 1 : (t + delta) >> 1; }
    constexpr int width() const { return a() + b() + 1; }
    constexpr int fb() const { return auto_bits(t + 1 - delta); }
    constexpr int hb() const { return columns ? auto_bits(width() - 1) : 0; }
    // bits of the characters in an entry's place (more than the width if the state's fields need it)
    constexpr int mb() const { return width() > fb() + hb() ? width() : fb() + hb(); }
};

struct AutoStates {
    static constexpr int kMost = 80;
    int n = 0;
    uint16_t code[kMost] = {};                   // the row's values, base 6
    uint8_t next[kMost][1 << kAutoWidth] = {};   // by the width() bits of equal characters
    uint8_t init[kAutoWidth + 1] = {};           // row 0 with 0, 1, .. positions (columns)
    uint8_t last[kMost] = {};                    // min(D(B), t + 1) - delta
    uint8_t top[kMost] = {};                     // largest band index with D <= t
};

// State 0 is the dead one (every value above t).
constexpr AutoStates auto_states(AutoShape S)
{
    AutoStates R;
    const int W = S.width(), t = S.t, B = S.b(), A = S.a();
    int16_t id[7776] = {};                       // code -> state + 1
    auto intern = [&](const int* d) {
        int code = 0;
        for (int k = W - 1; k >= 0; --k) code = code * 6 + d[k];
        if (!id[code]) {
            R.code[R.n] = (uint16_t)code;
            R.last[R.n] = (uint8_t)(d[B] - S.delta);
            for (int k = 0; k < W; ++k)
                if (d[k] <= t) R.top[R.n] = (uint8_t)k;
            id[code] = (int16_t)(++R.n);
        }
        return (uint8_t)(id[code] - 1);
    };
    int d[kAutoWidth] = {};
    for (int k = 0; k < W; ++k) d[k] = t + 1;
    intern(d);
    for (int positions = 0; positions <= B; ++positions) {
        for (int k = 0; k < W; ++k) {
            const int p = k - A, e = p + (k < B ? B - k : k - B);
            d[k] = p >= 0 && p <= positions && e <= t ? e : t + 1;
        }
        R.init[positions] = intern(d);
    }
    for (int s = 0; s < R.n; ++s) {
        int o[kAutoWidth] = {};
        int c = R.code[s];
        for (int k = 0; k < W; ++k) {
            o[k] = c % 6;
            c /= 6;
        }
        for (int m = 0; m < 1 << W; ++m) {
            int left = t + 1;
            for (int k = 0; k < W; ++k) {
                int v = o[k] + ((m >> k) & 1 ? 0 : 1);
                if (k + 1 < W) {
                    const int up = o[k + 1] + (k < B ? 2 : 0);
                    v = up < v ? up : v;
                }
                if (k > 0) {
                    const int l = left + (k > B ? 2 : 0);
                    v = l < v ? l : v;
                }
                v = v > t + 1 ? t + 1 : v;
                d[k] = left = v;
            }
            R.next[s][m] = intern(d);
        }
    }
    return R;
}

template <int T, int DELTA, int COLUMNS>
struct AutoFor {
    static constexpr AutoShape shape{T, DELTA, COLUMNS};
    static constexpr AutoStates states = auto_states(shape);
    static constexpr int bytes = states.n << (shape.mb() + 1);
};

// Cells of the band of Lemma 4 in the first s rows of a part of nr rows and nr + delta columns.
template <int T, int DELTA>
struct AutoCells {
    static constexpr int kMost = 48;             // rows 0 .. 47
    uint16_t cells[kMost][kMost] = {};           // [nr][s]
    constexpr AutoCells()
    {
        const int a = (T - DELTA) >> 1, b = (T + DELTA) >> 1;
        for (int nr = 0; nr < kMost; ++nr) {
            int sum = 0;
            for (int s = 1; s <= nr; ++s) {
                const int lo = s - a < 1 ? 1 : s - a, hi = s + b > nr + DELTA ? nr + DELTA : s + b;
                sum += hi - lo + 1;
                cells[nr][s] = (uint16_t)sum;
            }
        }
    }
};

// What a kernel needs to run a shape: 16 bytes, read as one.
struct alignas(16) AutoGeom {
    uint16_t init[kAutoWidth + 1];   // entry of row 0 with 0, 1, .. positions
    uint16_t dead;                   // entry of the dead state
    uint8_t a, fields;               // A; mb | fb << 4
};

// The tables of all shapes of thresholds up to TMAX, in one piece.  Offsets count from its start.
template <int TMAX>
struct AutoTable {
    static constexpr int kShapes = 2 * (TMAX + 1) * (TMAX + 1);
    static constexpr int index(int t, int delta, int columns)
    {
        return (t * (TMAX + 1) + delta) * 2 + columns;
    }
    template <int T, int DELTA, int COLUMNS>
    static constexpr int bytes_through()     // this shape's place and the ones before it
    {
        // equal lengths have one shape: steps over the rows
        constexpr bool here = DELTA <= T && !(DELTA == 0 && COLUMNS == 1);
        int before = 0;
        if constexpr (COLUMNS == 1) before = bytes_through<T, DELTA, 0>();
        else if constexpr (DELTA > 0) before = bytes_through<T, DELTA - 1, 1>();
        else if constexpr (T > 0) before = bytes_through<T - 1, T - 1, 1>();
        if constexpr (here) {
            constexpr int row = 2 << AutoFor<T, DELTA, COLUMNS>::shape.mb();
            return (before + row - 1) / row * row + AutoFor<T, DELTA, COLUMNS>::bytes;
        } else return before;
    }
    static constexpr int kBytes = (bytes_through<TMAX, TMAX, 1>() + 15) / 16 * 16;

    static constexpr int kCellRows = 48;

    alignas(16) uint16_t next[kBytes / 2];
    AutoGeom geom[kShapes];
    uint16_t cells[kShapes / 2 * kCellRows * kCellRows];   // [t][delta][nr][s]

    template <int T, int DELTA, int COLUMNS>
    constexpr void fill()
    {
        using F = AutoFor<T, DELTA, COLUMNS>;
        const int base = bytes_through<T, DELTA, COLUMNS>() - F::bytes;
        const int mb = F::shape.mb(), fb = F::shape.fb(), W = F::shape.width();
        auto entry = [&](int s) {
            return (uint16_t)(base + (s << (mb + 1)) + (F::states.last[s] << 1) +
                              (COLUMNS ? F::states.top[s] << (fb + 1) : 0));
        };
        for (int s = 0; s < F::states.n; ++s)
            for (int m = 0; m < 1 << mb; ++m)
                next[base / 2 + (s << mb) + m] = entry(F::states.next[s][m & ((1 << W) - 1)]);
        AutoGeom& g = geom[index(T, DELTA, COLUMNS)];
        for (int p = 0; p <= kAutoWidth; ++p)
            g.init[p] = entry(F::states.init[p < F::shape.b() ? p : F::shape.b()]);
        g.dead = entry(0);
        g.a = (uint8_t)F::shape.a();
        g.fields = (uint8_t)(mb | fb << 4);
        if (COLUMNS) return;
        constexpr AutoCells<T, DELTA> c;
        uint16_t* out = cells + index(T, DELTA, 0) / 2 * kCellRows * kCellRows;
        for (int nr = 0; nr < kCellRows; ++nr)
            for (int k = 0; k < kCellRows; ++k) out[nr * kCellRows + k] = c.cells[nr][k];
    }
    template <int T, int DELTA>
    constexpr void fill_from()
    {
        fill<T, DELTA, 0>();
        if constexpr (DELTA > 0) fill<T, DELTA, 1>();
        if constexpr (DELTA > 0) fill_from<T, DELTA - 1>();
        else if constexpr (T > 0) fill_from<T - 1, T - 1>();
    }
    constexpr AutoTable() : next{}, geom{}, cells{} { fill_from<TMAX, TMAX>(); }
};

}  // namespace pj

// lds_layout.hpp -- where the row FFT's LDS exchanges put each element.
//
// Stage s of a plan writes its butterfly outputs to the Stockham positions
// p = B + r Ns (B = (j - k) R + k, k = j mod Ns, r < R) and stage s + 1 reads
// p = t + m T (m < E).  Exchange s stores element p at f_s(p):
//  * a linear layout f(p) = p + p / P (P = 0: f(p) = p) with a padding period
//    P that keeps both sides affine in r and m -- P divides Ns, or Ns R
//    divides P (then B and B + (R - 1) Ns lie in one period), and P divides T
//    -- so that a thread forms one address per butterfly and one per read
//    sweep, the rest being immediate offsets;
//  * otherwise the fixed layout p + (p >> sh), whose addresses are formed
//    element by element.
// The period is chosen at compile time per exchange: the fewest LDS bank
// conflicts of a wave's writes and reads (64 banks of 4 bytes assumed; a
// half wave's elements counted per bank group), at no more LDS than the fixed
// layout, preferring its period 2^sh, then no padding, then the longest
// period; the fixed layout only where every linear one conflicts more.
// Host-compilable (constexpr only), so that the choice can be listed and
// tested on the CPU.
#pragma once

#include "fft_plan.hpp"

namespace scint {

// LDS layout of a row in the fixed scheme: one padding slot every 32
// elements breaks the power-of-two strides of the Stockham writes across
// banks.  A row whose padded length would not fit the 160 KB of LDS (20000
// complex64), or would just miss the 80 KB that lets two workgroups share a
// CU (10000), takes one slot every 64 elements.
#ifndef SCINT_LDS_PAD_SHIFT
#define SCINT_LDS_PAD_SHIFT 5
#endif
constexpr int kLdsPadShift = SCINT_LDS_PAD_SHIFT;
template <int L> constexpr int lds_pad_shift() {
    if (kLdsPadShift <= 0 || kLdsPadShift >= 6) return kLdsPadShift;
    const int b = (L + (L >> kLdsPadShift)) * 8, b6 = (L + (L >> 6)) * 8;
    return (b > 160 * 1024 || (b > 80 * 1024 && b6 <= 80 * 1024)) ? 6 : kLdsPadShift;
}
template <int L> constexpr int fixed_layout_length() {
    return lds_pad_shift<L>() > 0 ? L + (L >> lds_pad_shift<L>()) : L;
}

struct ExchLayout {
    bool linear;  // false: p + (p >> sh)
    int P;        // linear: p + p / P (0: p)
    int length;   // elements the exchange occupies
};

constexpr int layout_at(const ExchLayout &lay, int sh, int p) {
    return lay.linear ? (lay.P > 0 ? p + p / lay.P : p) : (sh > 0 ? p + (p >> sh) : p);
}

// Bank-conflict degree of one wave's access: the largest number of lanes of
// a half wave whose elements fall in the same group of banks (elements of
// elem_bytes, 64 banks of 4 bytes).
template <int N> constexpr int conflict_degree(const int (&addr)[N], int n, int elem_bytes) {
    const int groups = 256 / elem_bytes;
    int worst = 0;
    for (int h = 0; h < n; h += 32) {
        int cnt[64] = {};
        for (int i = h; i < n && i < h + 32; ++i) {
            const int g = addr[i] % groups;
            if (++cnt[g] > worst) worst = cnt[g];
        }
    }
    return worst;
}

template <int L, int V> constexpr int exch_conflicts(const ExchLayout &lay, int s, int elem_bytes, int rows = 1) {
    using P = Plan<L, V>;
    const int T = P::T, R = P::R[s], Ns = stage_ns<L, V>(s), sh = lds_pad_shift<L>();
    const int n = T * rows < 64 ? T * rows : 64;  // lane l: thread l / rows of row l % rows
    int worst = 0;
    int a[64] = {};
    for (int r = 0; r < 2 && r < R; ++r) {  // writes of butterflies j = t, outputs r
        for (int l = 0; l < n; ++l) {
            const int t = l / rows, k = t % Ns;
            a[l] = layout_at(lay, sh, (t - k) * R + k + r * Ns) * rows + l % rows;
        }
        const int c = conflict_degree(a, n, elem_bytes);
        if (c > worst) worst = c;
    }
    for (int l = 0; l < n; ++l) a[l] = layout_at(lay, sh, l / rows) * rows + l % rows;  // reads, m = 0
    const int c = conflict_degree(a, n, elem_bytes);
    return c > worst ? c : worst;
}

template <int L, int V> constexpr bool linear_ok(int s, int Pd) {
    using P = Plan<L, V>;
    const int T = P::T, R = P::R[s], Ns = stage_ns<L, V>(s);
    if (Pd == 0) return true;
    return (Ns % Pd == 0 || Pd % (Ns * R) == 0) && T % Pd == 0;
}

// The layout of exchange s (0 <= s < NS - 1) for elements of elem_bytes, with
// `rows` rows interleaved (element p of row b at f(p) rows + b; 1: a row on
// its own).
template <int L, int V> constexpr ExchLayout exch_layout(int s, int elem_bytes, int rows = 1) {
    using P = Plan<L, V>;
    const int T = P::T, sh = lds_pad_shift<L>(), limit = fixed_layout_length<L>();
    ExchLayout best{false, 0, limit};
    int best_c = exch_conflicts<L, V>(best, s, elem_bytes, rows);
    bool have_linear = false;
    auto consider = [&](int Pd) {
        if (!linear_ok<L, V>(s, Pd)) return;
        const int len = Pd > 0 ? L + L / Pd : L;
        if (len > limit) return;
        const ExchLayout cand{true, Pd, len};
        const int c = exch_conflicts<L, V>(cand, s, elem_bytes, rows);
        if (c < best_c || (c == best_c && !have_linear)) {
            best = cand;
            best_c = c;
            have_linear = true;
        }
    };
    if (sh > 0) consider(1 << sh);
    consider(0);
    for (int Pd = T; Pd >= 2; --Pd)
        if (T % Pd == 0) consider(Pd);
    return best;
}

// Elements a row's exchange buffer takes: the largest exchange layout.
template <int L, int V> constexpr int exch_buffer_length(int elem_bytes, int rows = 1) {
    int len = L;
    for (int s = 0; s + 1 < Plan<L, V>::NS; ++s) {
        const int l = exch_layout<L, V>(s, elem_bytes, rows).length;
        if (l > len) len = l;
    }
    return len;
}

// ---------------------------------------------------------------- columns
// Passes that hand their result to a pass along the other axis store it by
// columns up to 4096, so that no transpose runs between the two: the workgroup
// interleaves a few rows in its lanes (lane l is thread l / rows of row
// l % rows), and each element's store is a run of rows x elem_bytes.  Runs of
// 32 bytes meet in the L2 when the workgroups that share their lines run next
// to each other on one XCD; that needs rows small enough for four of them in
// the LDS.  Longer rows fit two at most, and runs of 16 bytes leave the L2
// before their line is whole (8192: 1.4 TB/s in the first propagation pass,
// 3.08 ms for 8 wavelengths against 2.5 ms with the transposes beside it), so
// from 5000 on the transposes stay.
constexpr int kColumnsMaxL = 4096;
constexpr bool stores_columns(int L) { return L <= kColumnsMaxL; }

// The smear's middle pass keeps a second row in its registers, which four rows
// of 4000 in one workgroup leave no room for: its passes keep the transposes
// from 4000 on (8 x 4000^2 x 4 disks: 2.93 ms by columns, 2.69 with them; 2560:
// 0.92 and 1.11).
constexpr int kSmearColumnsMaxL = 2560;
constexpr bool smear_columns(int L) { return L <= kSmearColumnsMaxL; }

// Real arrays are read and written by columns too while they stay in cache;
// above, runs half as long cost more than their transpose (2048: 140 us more
// in a pass over 16 patterns, transpose 84-104 us).
constexpr int kRealColumnsMaxL = 1024;
constexpr bool real_columns(int L) { return L <= kRealColumnsMaxL; }

// Rows that such a workgroup interleaves: up to four, runs of 32 bytes in FP32
// (16 x 2048^2 forward + adjoint: 1.97 ms; 16 bytes 2.26, 64 bytes 2.24 ms,
// whose 1024-thread workgroups fill a CU alone) and 64 in FP64, fewer where the
// LDS would hold one workgroup only, and fewer at the small sizes, whose rows
// would not occupy the chip.  Where the threads of a row divide a wave, at
// least a whole wave of them: 32 threads gave single calls the same time and
// batches half the rate (327 x 320^2 adjoints 458 us with two rows, 361 with
// four; 8192 x 64^2 FP64 screens 930 and 553 us).  Rows of 10 and 20 threads do
// not fill whole waves with more rows either: 100 keeps 40 threads, and 200 and
// 400 do in FP64 (26 x 400^2 screens 129 us, 139 with 80 threads).  16, a thread
// per row, keeps 32 (kept fields of 16384 FP64 screens 86 us, 131 with 64).
// Passes of two or more transforms outside a wavelength loop (heavy: screen +
// propagation, the adjoint's first) keep so many registers at 20 elements per
// thread that a CU holds 8 waves: from 2000 on they take as many rows as let
// two workgroups share it, since one alone waits at each of its barriers
// (adjoint from the kept field of 2 x 4000^2: 460 us with transposes, 500 with
// four rows, 471 with one; of 5 x 2560^2 446, 468, and 421 with two; FP64 screen
// + pattern of 5 x 2560^2 1665, 1702 with two, 1514 with one).
constexpr bool heavy_columns(int L, int E) { return L >= 2000 && E % 16 != 0; }

template <int L, int V> constexpr int column_rows(int elem_bytes, bool heavy = false) {
    const int T = Plan<L, V>::T;
    const bool whole = 64 % T == 0 || T % 64 == 0;
    const int least = whole || elem_bytes == 8 ? 60 : 120;  // of a row's length per row
    int rows = 1;
    while (2 * rows <= 4 && 2 * rows * least <= L) rows *= 2;
    while (T * rows < (64 % T == 0 && T > 1 ? 64 : 32)) rows *= 2;
    while (rows > 1 && (T * rows > 1024 || rows * exch_buffer_length<L, V>(elem_bytes, rows) * elem_bytes >
                                               (rows * elem_bytes > 32 ? 80 : 160) * 1024))
        rows /= 2;
    if (heavy && heavy_columns(L, Plan<L, V>::E))
        while (rows > 1 && (2 * ((T * rows + 63) / 64) > 8 ||
                            2 * rows * exch_buffer_length<L, V>(elem_bytes, rows) * elem_bytes > 160 * 1024))
            rows /= 2;
    return rows;
}

// Between 240 and 480, where two rows are more than half a wave (256, and 400 in
// FP32), a call on few rows takes two per workgroup (0: no such rule), twice the
// workgroups for a chip that they do not fill: up to 512 rows of 256 (one FP64
// screen + pattern 21.8 us, 22.6 with four rows; four of them 27.7 and 25.2), up
// to 8192 of 400, whose 80 threads fill a wave and a quarter (four screens +
// patterns 45.7 and 49.8 us; 209 adjoints from the kept field 440 and 380).
template <int L, int V> constexpr int few_column_limit() { return Plan<L, V>::T % 64 == 0 ? 512 : 8192; }
template <int L, int V> constexpr int few_column_rows(int elem_bytes) {
    return L >= 240 && L < 480 && 2 * Plan<L, V>::T > 32 && column_rows<L, V>(elem_bytes) > 2 ? 2 : 0;
}

// The first pass over several wavelengths (poly) writes that many fields.  Up to
// 320, where they are more than the 256 MB cache holds, its runs go to memory
// as they are: whole lines of 128 bytes, within 512 threads (11 wavelengths of
// 8192 x 64^2 screens 2.47 ms with transposes, 2.72 with runs of 32 bytes, 1.84
// with whole lines; of 512 x 256^2 2.39, 2.88 and 2.14).
constexpr int kPolyColumnsMaxL = 320;
constexpr long long kPolyCacheBytes = 256ll << 20;
template <int L, int V> constexpr int poly_column_rows(int elem_bytes) {
    const int T = Plan<L, V>::T;
    int rows = column_rows<L, V>(elem_bytes);
    if (L > kPolyColumnsMaxL || (64 % T != 0 && T % 64 != 0)) return rows;
    while (rows * elem_bytes < 128 && 2 * T * rows <= 512) rows *= 2;
    return rows;
}

// Row group and part (of `parts` workgroups that share a group's loop
// iterations) of workgroup w.  Workgroup w runs on XCD w % 8: the `line` row
// groups that share cache lines of what they store go to one XCD, next to each
// other in time, so that the parts of a line meet in its L2.
struct ColumnSlot {
    int group, part;
};
constexpr ColumnSlot column_slot(int w, int line, int parts) {
    const int q = w >> 3, set = q / line / parts;
    return ColumnSlot{(set * 8 + (w & 7)) * line + q % line, q / line % parts};
}

// Rows of one launch whose workgroups of `threads` take `rows` rows each, `parts`
// of them per group, in whole sets of `set` groups: a grid's threads are counted
// in 32 bits.
constexpr long long rows_per_launch(int threads, int rows, int set, long long parts) {
    return ((1ll << 32) - 1) / threads / parts / set * set * rows;
}

// Elements from one row of such a field to the next.  Stores by columns step
// by whole rows: whole lines of 128 bytes, and 13 lines more from 2000 on,
// which spreads them over the channels of the L2 (runs of 32 bytes written
// alone: 4096 2.3 -> 4.5 TB/s, 2048 3.5 -> 3.9, 2000 2.3 -> 2.9, 2560
// 4.0 -> 4.4; one line more is the worst choice at 2048, 1.8).
constexpr int field_pitch(int L, int elem_bytes) {
    const int line = 128 / elem_bytes;
    return stores_columns(L) ? (L + line - 1) / line * line + (L >= 2000 ? 13 * line : 0) : L;
}

}  // namespace scint

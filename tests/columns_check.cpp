// Host check of the sizes that store their fields by columns (lds_layout.hpp),
// built and run by tests/test_columns_host.py: the exchanges of interleaved
// rows map every element of every row to a slot of its own inside the buffer,
// the fields' rows hold a row, and the workgroups of a launch take every row
// group and part once.
#include <cstdio>
#include <vector>

#include "lds_layout.hpp"

using namespace scint;

static int failures = 0;
static void fail(const char *what, int L, int V, int eb) {
    std::printf("FAIL %s L=%d V=%d eb=%d\n", what, L, V, eb);
    ++failures;
}

template <int L, int V> static void check(int eb) {
    if (!stores_columns(L)) return;
    using P = Plan<L, V>;
    const int W = column_rows<L, V>(eb), buf = exch_buffer_length<L, V>(eb, W), sh = lds_pad_shift<L>();
    if (W < 1 || P::T * W > 1024 || (long long)W * buf * eb > 160 * 1024) fail("workgroup", L, V, eb);
    if (field_pitch(L, eb) < L || field_pitch(L, eb) * eb % 128) fail("pitch", L, V, eb);
    for (int s = 0; s + 1 < P::NS; ++s) {
        const ExchLayout lay = exch_layout<L, V>(s, eb, W);
        const int R = P::R[s], Ns = stage_ns<L, V>(s);
        std::vector<char> used((size_t)W * buf, 0);
        for (int b = 0; b < W; ++b)
            for (int p = 0; p < L; ++p) {
                const int a = layout_at(lay, sh, p) * W + b;
                if (a < 0 || a >= W * buf || used[a]) return fail("slot", L, V, eb);
                used[a] = 1;
            }
        if (!lay.linear) continue;
        const int ws = Ns + ((lay.P > 0 && Ns % lay.P == 0) ? Ns / lay.P : 0), rs = P::T + (lay.P > 0 ? P::T / lay.P : 0);
        for (int j = 0; j < L / R; ++j) {
            const int k = j % Ns, base = (j - k) * R + k, q = lay.P > 0 ? base + base / lay.P : base;
            for (int r = 0; r < R; ++r)
                if (q + r * ws != layout_at(lay, sh, base + r * Ns)) return fail("write", L, V, eb);
        }
        for (int t = 0; t < P::T; ++t) {
            const int q = lay.P > 0 ? t + t / lay.P : t;
            for (int m = 0; m < P::E; ++m)
                if (q + m * rs != layout_at(lay, sh, t + m * P::T)) return fail("read", L, V, eb);
        }
    }
    std::printf("ok L=%d V=%d eb=%d rows=%d\n", L, V, eb, W);
}

static void check_slots(int line, int groups, int parts) {
    const int set = 8 * line, grid = (groups + set - 1) / set * set * parts;
    std::vector<int> seen((size_t)groups * parts, 0);
    for (int w = 0; w < grid; ++w) {
        const ColumnSlot c = column_slot(w, line, parts);
        if (c.part < 0 || c.part >= parts || c.group < 0) return fail("slot range", line, groups, parts);
        if (c.group < groups) ++seen[(size_t)c.group * parts + c.part];
    }
    for (int n : seen)
        if (n != 1) return fail("slot cover", line, groups, parts);
}

int main() {
#define SCINT_F64_CASE(LL) check<LL, 0>(16), check<LL, 0>(8);
    SCINT_SIZES_F64(SCINT_F64_CASE)
#define SCINT_V_CASE(LL, VV) check<LL, VV>(8);
    SCINT_VARIANTS_F32(SCINT_V_CASE)
    for (int line : {1, 2, 4, 8})
        for (int groups : {1, 5, 8, 25, 64, 333, 1000})
            for (int parts : {1, 2, 3, 7}) check_slots(line, groups, parts);
    std::printf("%d failures\n", failures);
    return failures ? 1 : 0;
}

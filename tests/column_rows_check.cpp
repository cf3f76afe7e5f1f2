// Host check of the rows that a workgroup of the passes by columns interleaves
// (lds_layout.hpp), built and run by tests/test_column_rows_host.py: whole waves
// where the threads of a row divide one, within the limits of a workgroup, and
// the exchanges of every element in a slot of its own.
#include <cstdio>
#include <vector>

#include "lds_layout.hpp"

using namespace scint;

static int failures = 0;

template <int L, int V> static bool slots_ok(int eb, int W) {
    using P = Plan<L, V>;
    const int buf = exch_buffer_length<L, V>(eb, W), sh = lds_pad_shift<L>();
    if (W < 1 || P::T * W > 1024 || (long long)W * buf * eb > 160 * 1024) return false;
    for (int s = 0; s + 1 < P::NS; ++s) {
        const ExchLayout lay = exch_layout<L, V>(s, eb, W);
        std::vector<char> used((size_t)W * buf, 0);
        for (int b = 0; b < W; ++b)
            for (int p = 0; p < L; ++p) {
                const int a = layout_at(lay, sh, p) * W + b;
                if (a < 0 || a >= W * buf || used[a]) return false;
                used[a] = 1;
            }
    }
    return true;
}

template <int L, int V> static void check(int eb) {
    if (!stores_columns(L)) return;
    const int T = Plan<L, V>::T, W = column_rows<L, V>(eb);
    bool ok = slots_ok<L, V>(eb, W);
    if (64 % T == 0 && T > 1 && T * W % 64 != 0) ok = false;  // an unfilled wave
    // the passes of many transforms: two workgroups on a CU at the sizes that ask for it
    const int H = column_rows<L, V>(eb, true);
    ok = ok && slots_ok<L, V>(eb, H) && H <= W;
    if (heavy_columns(L, Plan<L, V>::E)) {
        if (2 * ((T * H + 63) / 64) > 8 || 2 * H * exch_buffer_length<L, V>(eb, H) * eb > 160 * 1024) ok = false;
    } else if (H != W) {
        ok = false;
    }
    // calls on few rows
    const int Z = few_column_rows<L, V>(eb);
    ok = ok && (Z == 0 || (Z < W && slots_ok<L, V>(eb, Z)));
    // the first pass over many wavelengths
    const int Q = poly_column_rows<L, V>(eb);
    ok = ok && slots_ok<L, V>(eb, Q) && Q >= W && (Q == W || (L <= kPolyColumnsMaxL && T * Q <= 512));
    std::printf("%s L=%d V=%d eb=%d threads per row %d, rows %d, %d, %d\n", ok ? "ok" : "FAIL", L, V, eb, T, W, H, Q);
    failures += !ok;
}

// launches of more rows than a grid's 32-bit thread count allows are cut
static void check_launches() {
    for (int threads : {32, 64, 250, 256, 1000, 1024})
        for (int rows : {1, 2, 4, 64, 256})
            for (int set : {8, 64, 128})
                for (long long parts : {1, 2, 7, 64}) {
                    const long long most = rows_per_launch(threads, rows, set, parts);
                    const long long grid = (most / rows + set - 1) / set * set * parts;
                    const bool ok = most >= (long long)rows * set && most % ((long long)rows * set) == 0 &&
                                    grid * threads < (1ll << 32) && most + (long long)rows * set * 2 > ((1ll << 32) - 1) / threads / parts * rows;
                    if (!ok) std::printf("FAIL threads=%d rows=%d set=%d parts=%lld: %lld\n", threads, rows, set, parts, most);
                    failures += !ok;
                }
}

int main() {
    check_launches();
#define SCINT_F64_CASE(LL) check<LL, f64_plan(LL)>(16), check<LL, 0>(8);
    SCINT_SIZES_F64(SCINT_F64_CASE)
#define SCINT_V_CASE(LL, VV) check<LL, VV>(8);
    SCINT_VARIANTS_F32(SCINT_V_CASE)
    std::printf("%d failures\n", failures);
    return failures ? 1 : 0;
}

// row_inst.hip -- explicit instances of the row-pass kernel for one precision
// and one program, selected at compile time by SCINT_REAL and SCINT_PROG
// (the build compiles this file once per pair).
#include "row_kernel.hpp"
#include "row_launch.h"

#include <algorithm>

#ifndef SCINT_REAL
#error "SCINT_REAL (float or double) must be defined"
#endif
#ifndef SCINT_PROG
#error "SCINT_PROG (a program name such as ProgNoise) must be defined"
#endif

#define SCINT_CAT2(a, b) a##b
#define SCINT_CAT(a, b) SCINT_CAT2(a, b)

namespace scint {

// W rows interleaved in a workgroup (0: none)
template <int L, int V, int W>
static hipError_t launch_rows(const RowProgram &prog, const void *tw, hipStream_t stream) {
    using Cfg = RowCfg<SCINT_REAL, L, V, W>;
    // passes that store by columns need no transposes beside them, and only the
    // sizes of real_columns take phase screens by columns
    constexpr bool smear = std::is_same<SCINT_PROG, ProgSmearFwdT>::value ||
                           std::is_same<SCINT_PROG, ProgSmearMidT>::value || std::is_same<SCINT_PROG, ProgInvReT>::value;
    constexpr bool wanted = !(has_side<SCINT_PROG>() && (smear ? smear_columns(L) : stores_columns(L))) &&
                            (real_columns(L) || !std::is_same<SCINT_PROG, ProgPhasePropX>::value);
    if constexpr (!wanted) {
        return hipErrorInvalidValue;
    } else {
    RowProgram p = prog;
    if constexpr (Cfg::IL) {
        // whole sets of 8 XCDs x LINE_GROUPS row groups (row_kernel)
        const int64_t set = 8 * Cfg::LINE_GROUPS, groups = (prog.total_rows - prog.row0 + Cfg::B - 1) / Cfg::B;
        p.iter_split = iter_splittable<SCINT_PROG>() ? std::min(std::max(prog.iter_split, 1), prog.n_iter) : 1;
        const int64_t grid = (groups + set - 1) / set * set * p.iter_split;
        if (grid > (1ll << 31) - 1) return hipErrorInvalidValue;
        hipLaunchKernelGGL((row_kernel<SCINT_REAL, L, V, SCINT_PROG, W>), dim3((unsigned)grid), dim3(Cfg::THREADS), 0,
                           stream, p, static_cast<const cpx<SCINT_REAL> *>(tw));
        return hipGetLastError();
    }
    // two workgroups per row only where the program allows it, the loop has
    // two or more iterations and the row workgroups come in whole eights
    const int row_wgs = (prog.total_rows - prog.row0 + Cfg::B - 1) / Cfg::B;
    p.iter_split = !iter_splittable<SCINT_PROG>() || prog.n_iter < 2   ? 1
                   : prog.iter_split > 2 && !has_side<SCINT_PROG>()     ? std::min(prog.iter_split, prog.n_iter)
                   : prog.iter_split >= 2 && row_wgs % 8 == 0           ? 2
                                                                        : 1;
    if (p.iter_split == 2 && row_wgs % 8 != 0) p.iter_split = 1;
    const int rows_blocks = row_wgs * p.iter_split;
    if constexpr (has_side<SCINT_PROG>()) {
        // groups of fft_blocks row workgroups and side_blocks transpose
        // workgroups; the units are spread evenly over the latter
        RowSide &sd = p.side;
        const int64_t units = sd.u1 - sd.u0;
        if (sd.fft_blocks < 1 || sd.side_blocks < 1 || units < 1 || sd.u0 < 0 || !sd.in || !sd.out)
            return hipErrorInvalidValue;
        sd.groups = (rows_blocks + sd.fft_blocks - 1) / sd.fft_blocks;
        const int64_t nside = (int64_t)sd.groups * sd.side_blocks;
        const int64_t per = (units + nside - 1) / nside;
        if (per > (1 << 30) || (int64_t)sd.groups * (sd.fft_blocks + sd.side_blocks) > (1ll << 31) - 1)
            return hipErrorInvalidValue;
        sd.units_per_block = (int32_t)per;
        const int grid = sd.groups * (sd.fft_blocks + sd.side_blocks);
        hipLaunchKernelGGL((row_kernel<SCINT_REAL, L, V, SCINT_PROG, W>), dim3(grid), dim3(Cfg::THREADS), 0, stream, p,
                           static_cast<const cpx<SCINT_REAL> *>(tw));
    } else {
        hipLaunchKernelGGL((row_kernel<SCINT_REAL, L, V, SCINT_PROG, W>), dim3(rows_blocks), dim3(Cfg::THREADS), 0,
                           stream, p, static_cast<const cpx<SCINT_REAL> *>(tw));
    }
    return hipGetLastError();
    }
}

// the same in pieces of whole sets of row groups, as many rows as the threads
// of a launch can be counted for
template <int L, int V, int W>
static hipError_t launch_pieces(const RowProgram &prog, const void *tw, hipStream_t stream) {
    using Cfg = RowCfg<SCINT_REAL, L, V, W>;
    const int64_t parts = iter_splittable<SCINT_PROG>() ? std::min(std::max(prog.iter_split, 1), prog.n_iter) : 1;
    const int64_t most = rows_per_launch(Cfg::THREADS, Cfg::B, Cfg::IL ? 8 * Cfg::LINE_GROUPS : 8, parts);
    if (has_side<SCINT_PROG>() || prog.total_rows - prog.row0 <= most) return launch_rows<L, V, W>(prog, tw, stream);
    RowProgram p = prog;
    for (int64_t r = prog.row0; r < prog.total_rows; r += most) {
        p.row0 = (int32_t)r;
        p.total_rows = (int32_t)std::min<int64_t>(r + most, prog.total_rows);
        if (hipError_t e = launch_rows<L, V, W>(p, tw, stream)) return e;
    }
    return hipSuccess;
}

template <int L, int V>
static hipError_t launch_one(const RowProgram &prog, const void *tw, hipStream_t stream) {
    constexpr int W = program_rows<SCINT_REAL, L, V, SCINT_PROG>(), elem = 2 * (int)sizeof(SCINT_REAL);
    if constexpr (W > 0) {
        constexpr int WF = few_column_rows<L, V>(elem);
        if constexpr (WF > 0)
            if (prog.total_rows - prog.row0 <= few_column_limit<L, V>()) return launch_pieces<L, V, WF>(prog, tw, stream);
    }
    if constexpr (std::is_same<SCINT_PROG, ProgPhaseProp>::value && stores_columns(L)) {
        constexpr int WP = poly_column_rows<L, V>(elem);
        const int64_t bytes = (int64_t)(prog.total_rows - prog.row0) * prog.n_iter * field_pitch(L, elem) * elem;
        if (WP != W && bytes > kPolyCacheBytes) return launch_pieces<L, V, WP>(prog, tw, stream);
    }
    return launch_pieces<L, V, W>(prog, tw, stream);
}

template <>
hipError_t launch_row<SCINT_REAL, SCINT_CAT(SCINT_PROG, Tag)>(int L, int V, const RowProgram &prog, const void *tw,
                                                               hipStream_t stream) {
#define SCINT_CASE(LL) \
    case LL:           \
        if (V == 0) return launch_one<LL, SCINT_IS_F64 ? f64_plan(LL) : 0>(prog, tw, stream); \
        break;
#define SCINT_VCASE(LL, VV) \
    if (L == LL && V == VV) return launch_one<LL, VV>(prog, tw, stream);
#if !SCINT_IS_F64
    SCINT_VARIANTS_F32(SCINT_VCASE)
#endif
    switch (L) {
#if SCINT_IS_F64
        SCINT_SIZES_F64(SCINT_CASE)
#else
        SCINT_SIZES_F32(SCINT_CASE)
#endif
    default:
        break;
    }
    return hipErrorInvalidValue;
#undef SCINT_CASE
#undef SCINT_VCASE
}

}  // namespace scint

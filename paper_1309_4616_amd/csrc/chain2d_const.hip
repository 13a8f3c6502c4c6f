// Chain sweeps of 2D constant-coefficient stencils (chain2d.h).
#include <algorithm>

#include "chain2d.h"

namespace expi {

hipError_t launch_chain2d_var(int coef, int tw, int vec, int n, int grid, const ChainArgs& a, hipStream_t s);

namespace {

hipError_t launch_const(int vec, bool stream, int n, int grid, const ChainArgs& a, hipStream_t s) {
    using namespace chain;
    if (stream) {
        if (n == 2) return go<double, 2, 2, C_CONST, true>(grid, a, s);
        if (n == 4) return go<double, 2, 4, C_CONST, true>(grid, a, s);
        if (n == 5) return go<double, 2, 5, C_CONST, true>(grid, a, s);
        if (n == 6) return go<double, 2, 6, C_CONST, true>(grid, a, s);
    }
    if (n == 2) return vec == 2 ? go<double, 2, 2, C_CONST>(grid, a, s) : go<double, 1, 2, C_CONST>(grid, a, s);
    if (n == 4) return vec == 2 ? go<double, 2, 4, C_CONST>(grid, a, s) : go<double, 1, 4, C_CONST>(grid, a, s);
    if (n == 5) return vec == 2 ? go<double, 2, 5, C_CONST>(grid, a, s) : go<double, 1, 5, C_CONST>(grid, a, s);
    if (n == 6) return vec == 2 ? go<double, 2, 6, C_CONST>(grid, a, s) : go<double, 1, 6, C_CONST>(grid, a, s);
    return hipErrorInvalidValue;
}

}  // namespace

// Not the constant coefficient with FP32 storage: its pair sweep
// (pair2d.hip) rounds a row's diagonal in one or two operations depending on
// the row's place in its tile, so a chain would not reproduce its results to
// better than FP32 rounding (about 1e-7), which callers can see in the
// float64 result.  The other kinds round as their single product does.
bool chain2d_supported(const Op& op, int tw) {
    // buffer offsets are 32-bit byte offsets: below 2^31 bytes in FP64
    return op.kind == 0 && op.dim == 2 && op.size * 8 < ((int64_t)1 << 31) - 64 &&
           !(op.coef == EXPI_COEF_CONST && tw == 1);
}

// Products per chain: up to 6 with a constant coefficient, 2 and 4 with the
// others (the face weights
// of T + 1 rows take the registers that two more levels would need).
bool chain2d_length(const Op& op, int n) {
    return op.coef == EXPI_COEF_CONST ? (n == 2 || (n >= 4 && n <= 6)) : (n == 2 || n == 4);
}

// room: bytes the launch has for its partials; the grid is no larger than they
// hold (the waves stride over the tiles).  partials_bytes always has room for
// 256 workgroups, one wave per SIMD.
static ChainShape chain2d_shape(const Op& op, int n, int cus, bool aligned, size_t room) {
    ChainShape g{};
    const int fit = (int)std::min<size_t>(room / (chain::kStride * sizeof(double)), 1 << 20) / kXcd * kXcd;
    g.vec = (op.n[0] % 2 == 0 && aligned) ? 2 : 1;
    // streaming stores where the three vectors of a pass exceed the last-level
    // cache (256 MB): at 8192^2 they leave it to the rows read twice, 516 ->
    // 485 us per pass; on grids that fit, the next pass would miss what they
    // write (1500 x 1100: 19 -> 24 us with a stored coefficient)
    g.stream = op.coef == EXPI_COEF_CONST && g.vec == 2 && op.size * 24 > ((int64_t)256 << 20) && op.n[0] >= 512;
    const int hx = chain::halo_columns(n, g.vec, g.stream), out = 64 * g.vec - 2 * hx;
    g.tiles0 = op.n[0] <= 64 * g.vec ? 1 : (op.n[0] - 2 * hx + out - 1) / out;
    // rows per tile: as few tiles as fill the wave slots (two waves per SIMD)
    // once, so that every wave takes one tile and the rows loaded twice are
    // few; a multiple of the unrolled block
    const int u = chain::kRows;
    const int slots = std::min(2 * 4 * std::max(cus, kXcd), chain::kWaves * fit);
    const int bands = std::max(1, slots / g.tiles0);
    int march = (op.n[1] + bands - 1) / bands;
    march = (march + u - 1) / u * u;
    g.march = march;
    g.ntiles = g.tiles0 * ((op.n[1] + march - 1) / march);
    const int wgs = (g.ntiles + chain::kWaves - 1) / chain::kWaves;
    const int most = std::min(2 * std::max(cus, kXcd) / kXcd * kXcd, fit);
    g.grid = std::min(most, (wgs + kXcd - 1) / kXcd * kXcd);
    return g;
}

size_t chain2d_partials(const Op& op, int n, int cus, size_t room) {
    // whatever the points per lane turn out to be
    const int grid = std::max(chain2d_shape(op, n, cus, false, room).grid, chain2d_shape(op, n, cus, true, room).grid);
    return (size_t)grid * chain::kStride * sizeof(double);
}

hipError_t launch_chain2d(const Op& op, int tw, int n, ChainArgs a, int cus, size_t room, int* nparts,
                          hipStream_t s) {
    if (!chain2d_supported(op, tw) || !chain2d_length(op, n)) return hipErrorInvalidValue;
    for (int q = 0; q < 2; ++q) {
        a.n[q] = op.n[q];
        a.ih2[q] = 1.0 / (op.h[q] * op.h[q]);
        a.hpos[q] = op.h[q];
        a.c0ih[q] = op.c0 * a.ih2[q];
    }
    a.c0 = op.c0;
    a.c1 = op.c1;
    a.tx = op.tx;
    a.ty = op.ty;
    a.field = op.field;
    a.bc = op.bc;
    const size_t sz = tw == 1 ? 4 : 8;
    auto on = [&](size_t al) {
        return (uintptr_t)a.x % al == 0 && (uintptr_t)a.out % al == 0 && (uintptr_t)a.p % al == 0;
    };
    const bool fld = op.coef != EXPI_COEF_FIELD || (uintptr_t)op.field % 16 == 0;
    const ChainShape g = chain2d_shape(op, n, cus, on(2 * sz) && fld, room);
    if (g.grid < kXcd) return hipErrorInvalidValue;
    a.march = g.march;
    a.tiles0 = g.tiles0;
    a.ntiles = g.ntiles;
    *nparts = g.grid;
    return op.coef == EXPI_COEF_CONST ? launch_const(g.vec, g.stream, n, g.grid, a, s)
                                      : launch_chain2d_var(op.coef, tw, g.vec, n, g.grid, a, s);
}

}  // namespace expi

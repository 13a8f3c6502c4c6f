// Chain sweeps of 2D stencils with a position-dependent coefficient
// (chain2d.h): stored field, separable tables, D(x, y) times the Laplacian.
#include "chain2d.h"

namespace expi {
namespace {

template <class TW, int V, int T>
hipError_t pick(int coef, int grid, const ChainArgs& a, hipStream_t s) {
    using namespace chain;
    switch (coef) {
        case EXPI_COEF_FIELD: return go<TW, V, T, C_FIELD>(grid, a, s);
        case EXPI_COEF_SEPARABLE: return go<TW, V, T, C_SEP>(grid, a, s);
        case EXPI_COEF_DLAP: return go<TW, V, T, C_DLAP>(grid, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_chain2d_var(int coef, int tw, int vec, int n, int grid, const ChainArgs& a, hipStream_t s) {
    if (tw == 0) {
        if (n == 2) return vec == 2 ? pick<double, 2, 2>(coef, grid, a, s) : pick<double, 1, 2>(coef, grid, a, s);
        if (n == 4) return vec == 2 ? pick<double, 2, 4>(coef, grid, a, s) : pick<double, 1, 4>(coef, grid, a, s);
    } else {
        if (n == 2) return vec == 2 ? pick<float, 2, 2>(coef, grid, a, s) : pick<float, 1, 2>(coef, grid, a, s);
        if (n == 4) return vec == 2 ? pick<float, 2, 4>(coef, grid, a, s) : pick<float, 1, 4>(coef, grid, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace expi

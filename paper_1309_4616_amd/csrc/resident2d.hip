// A whole Newton loop of a small 2D constant-coefficient stencil in one
// launch of one workgroup (Sec. III-C: products, norms and two-term stop test
// until it holds), FP64.
//
// What bounds a small grid is latency: at 128^2 a pass over memory is a few
// microseconds of launch, march and stop test for 0.4 MB of data.  Here w and
// p stay in the registers of one workgroup of 8 waves (256 VGPRs each: up to
// 32 points per thread, 16,384 points in all) from the start vector to the
// stop; one product costs one exchange of the strips' edge rows through LDS
// and one barrier, and two products one sum of the waves' norms.  Measured per
// call: 128^2, degree 21: 72 us (the kernel 55), against 74 us in four chain
// sweeps and 123 us in pair sweeps; 100 x 37 over three substeps: 209 us
// against 351 and 719.  The products themselves bound it at 128^2 (2.6 us
// each on one CU), the chain of exchange, sums and test on small grids
// (1.2 us).  Grids with more points would
// need several workgroups to meet at every product, which costs more
// (6 us for 256 workgroups) than the chain sweeps' launches.
//
// Layout: a wave holds 64 V columns (V per lane) of R consecutive rows; CX
// waves side by side cover a row, 8 / CX such groups cover the rows.  The
// x neighbours come from the adjacent lanes by wave shifts, those beyond the
// wave and the rows above and below from LDS (two copies, used in turn).
// Points beyond the grid hold zero and have weight zero.  What fits: rows of
// up to 64 points with 24 rows per wave (192 rows), up to 128 points with 16
// (128 rows), and longer rows over CX waves with 12 rows per wave (129 to 256
// points: 48 rows; up to 1024: 12); edge columns and one point per lane take
// registers that more rows would need.
#include <algorithm>
#include <cmath>

#include "sweep_common.h"

namespace expi {
namespace {

constexpr int kResWaves = 8;
constexpr int kResMaxPoints = 32;   // points per thread (V R) at most

// v plus the value that CTRL brings in (0 where it brings none).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    if constexpr (ROWS == 0xF) return v + dpp_shift0<CTRL>(v);
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xF, false);
    return v + __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
// Sum over each row of 16 lanes, in its last lane.
__device__ __forceinline__ double row_sum(double v) {
    v = dpp_add<0x111, 0xF>(v);
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    return dpp_add<0x118, 0xF>(v);
}
// Sum over the wave, in lane 63 (row sums passed on by row broadcasts).
__device__ __forceinline__ double wave_sum_last(double v) {
    v = row_sum(v);
    v = dpp_add<0x142, 0xA>(v);
    return dpp_add<0x143, 0xC>(v);
}
__device__ __forceinline__ double lane_get(double v, int l) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// f(0), f(1), ... with constant arguments; the second kind stops at `n`.
template <int A, int B, class F>
__device__ __forceinline__ void for_rows(F& f) {
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        for_rows<A + 1, B>(f);
    }
}
template <int A, int B, class F>
__device__ __forceinline__ void for_rows_while(F& f, int n) {
    if constexpr (A < B) {
        if (A < n) {
            f(std::integral_constant<int, A>{});
            for_rows_while<A + 1, B>(f, n);
        }
    }
}

template <int V, int R, int C, bool WIDE, bool IO>
__global__ __launch_bounds__(kResWaves * 64, 1) void resident2d_loop(ResidentArgs a) {
    constexpr int WX = 64 * V;
    // edge rows of every wave (top, bottom) and edge columns (left, right)
    __shared__ double rows[2][kResWaves][2][WX];
    __shared__ double cols[2][WIDE ? kResWaves : 1][2][R];
    __shared__ double part[kResWaves][4];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = a.n[0], n1 = a.n[1];
    const int CX = WIDE ? a.cx : 1, RG = a.groups;   // WIDE: several waves per grid row
    const int cx = wv % CX, rg = wv / CX;
    const int x0 = cx * WX + lane * V;
    // rows dealt out evenly: n1 / RG or one more per group, R - C .. R of them
    const int base = n1 / RG, extra = n1 - base * RG;
    const int nr = rg < RG ? base + (rg < extra ? 1 : 0) : 0;
    const int y0 = rg * base + min(rg, extra);
    const bool top = y0 == 0, last = nr > 0 && y0 + nr == n1;
    const bool dir = (a.bc == EXPI_DIRICHLET0);
    double axm[V], axq[V], adx[V];
    bool in[V], xb[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int x = x0 + v;
        const bool em = x > 0, eq = x < n0 - 1;
        in[v] = x < n0;
        xb[v] = !(em && eq);
        axm[v] = in[v] && em ? a.afx : 0.0;
        axq[v] = in[v] && eq ? a.afx : 0.0;
        adx[v] = ((em || dir) ? a.afx : 0.0) + ((eq || dir) ? a.afx : 0.0);
    }
    double w[R][V], p[R][V];
    double s0 = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int y = y0 + r;
            w[r][v] = (r < nr && in[v]) ? a.x[(size_t)y * n0 + x0 + v] : 0.0;
            p[r][v] = 0.0;
            s0 += w[r][v] * w[r][v];
        }
    }
    // edges of the waves' strips for the next product (bot: the last row)
    double bot[V];
#pragma unroll
    for (int v = 0; v < V; ++v) bot[v] = w[0][v];
#pragma unroll
    for (int r = 1; r < R; ++r)
#pragma unroll
        for (int v = 0; v < V; ++v) bot[v] = r < nr ? w[r][v] : bot[v];
    auto publish = [&](int par) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            rows[par][wv][0][lane * V + v] = w[0][v];
            rows[par][wv][1][lane * V + v] = bot[v];
        }
        if constexpr (WIDE) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (lane == 0) cols[par][wv][0][r] = w[r][0];
                if (lane == 63) cols[par][wv][1][r] = w[r][V - 1];
            }
        }
    };
    // this wave's sums (written between two barriers that every reader of the
    // last ones has passed)
    auto sums = [&](double t0, double t1, double t2, double t3) __attribute__((always_inline)) {
        t0 = wave_sum_last(t0);
        t1 = wave_sum_last(t1);
        t2 = wave_sum_last(t2);
        t3 = wave_sum_last(t3);
        if (lane == 63) {
            part[wv][0] = t0;
            part[wv][1] = t1;
            part[wv][2] = t2;
            part[wv][3] = t3;
        }
    };
    // product j into w, p, and its sums
    auto product = [&](int j, double& s1, double& s2) __attribute__((always_inline)) {
        const int par = j & 1;
        const double beta = a.beta[j], d = a.d[j + 1];
        // (a strip at the grid's edge reads some other strip's row: weight 0)
        const int wu = rg > 0 ? wv - CX : wv, wd = min(wv + CX, kResWaves - 1);
        double prev[V], dn[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            prev[v] = rows[par][wu][1][lane * V + v];
            dn[v] = rows[par][wd][0][lane * V + v];
        }
        const double cd2 = minus<double>(beta, a.afy2), cd1 = minus<double>(beta, a.afy);
        auto row = [&](auto rc) __attribute__((always_inline)) {
            constexpr int r = decltype(rc)::value;
            // only a strip's first row and its last few can be at the grid's
            // edge: the others take their weights without a choice
            constexpr bool kEnd = r >= R - C - 1;
            const bool em = r > 0 || !top, eq = !kEnd || r < nr - 1 || !last;
            const double aym = em ? a.afy : 0.0, ayq = eq ? a.afy : 0.0;
            const bool cm = em || dir, cq = eq || dir;
            const double cdy = (cm && cq) ? cd2 : ((cm || cq) ? cd1 : beta);
            double left = dpp_shift0<kDppWaveShr1>(w[r][V - 1]);
            double right = dpp_shift0<kDppWaveShl1>(w[r][0]);
            if constexpr (WIDE) {
                if (lane == 0 && cx > 0) left = cols[par][wv - 1][1][r];
                if (lane == 63 && cx < CX - 1) right = cols[par][min(wv + 1, kResWaves - 1)][0][r];
            }
            double o[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const double wl = (v > 0) ? w[r][v - 1] : left;
                const double wr = (v < V - 1) ? w[r][v + 1] : right;
                const double below = w[r < R - 1 ? r + 1 : r][v];
                const double wq = !kEnd ? below : (r < nr - 1 ? below : dn[v]);
                o[v] = const_product<double>(axm[v], axq[v], aym, ayq, minus<double>(cdy, adx[v]), wl, wr, prev[v], wq,
                                             w[r][v]);
                if constexpr (IO) o[v] = (xb[v] || !(em && eq)) ? beta * w[r][v] : o[v];
            }
#pragma unroll
            for (int v = 0; v < V; ++v) {
                prev[v] = w[r][v];
                p[r][v] = (j == 0) ? __builtin_elementwise_fma(a.d[0], w[r][v], d * o[v])
                                   : __builtin_elementwise_fma(d, o[v], p[r][v]);
                w[r][v] = o[v];
                if constexpr (kEnd) bot[v] = o[v];
                s1 += o[v] * o[v];
                s2 += p[r][v] * p[r][v];
            }
        };
        // (waves without rows only keep the barriers)
        if (nr > 0) {
            for_rows<0, R - C>(row);
            for_rows_while<R - C, R>(row, nr);
        }
    };
    // square roots of the four sums over all waves, the same in every lane
    auto norms = [&](double (&n)[4]) __attribute__((always_inline)) {
        static_assert(kResWaves == 8, "eight values per group of lanes");
        double t = part[lane & 7][(lane >> 3) & 3];
        t = dpp_add<0x111, 0xF>(t);
        t = dpp_add<0x112, 0xF>(t);
        t = sqrt(dpp_add<0x114, 0xF>(t));   // lanes 7, 15, 23, 31: sums of their eight
#pragma unroll
        for (int q = 0; q < 4; ++q) n[q] = lane_get(t, 8 * q + 7);
    };
    sums(s0, 0.0, 0.0, 0.0);
    publish(0);
    __syncthreads();
    double n[4];
    norms(n);
    const double rn = n[0];
    double tprev = fabs(a.d[0]) * rn;
    const bool first = threadIdx.x == 0;
    if (first) {
        a.st->rnorm = a.mirror->rnorm = rn;
        a.st->hist[0] = a.mirror->hist[0] = tprev;
    }
    double wn = 0.0, pn = 0.0, num = 0.0;
    int done = 0, m = 0;
    // the two-term test at degree `deg`, the same in every wave (they all sum
    // the same values)
    auto test = [&](int deg, double wnorm, double pnorm) __attribute__((always_inline)) {
        const double t = fabs(a.d[deg]) * wnorm;
        m = deg;
        wn = wnorm;
        pn = pnorm;
        num = tprev + t;
        if (first && deg < kHist) a.st->hist[deg] = a.mirror->hist[deg] = t;
        if (!isfinite(wn) || !isfinite(pn) || !isfinite(tprev)) done = 2;
        else if (deg >= 2 && num <= a.tol * pn) done = 1;
        tprev = t;
        return __builtin_amdgcn_readfirstlane(done) != 0;
    };
    // two products per round: the sums of both go out at the second's
    // barrier, so the tests cost one exchange for two products; a stop at the
    // first takes the second one's term back out of p
#pragma unroll 1
    for (int j = 0; j < a.m_max; j += 2) {
        double s1 = 0.0, s2 = 0.0, s3 = 0.0, s4 = 0.0;
        product(j, s1, s2);
        publish(1);
        __syncthreads();
        const bool two = j + 1 < a.m_max;
        if (two) product(j + 1, s3, s4);
        sums(s1, s2, s3, s4);
        publish(0);
        __syncthreads();
        norms(n);
        if (test(j + 1, n[0], n[1])) {
            const double d2 = two ? a.d[j + 2] : 0.0;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int v = 0; v < V; ++v) p[r][v] = __builtin_elementwise_fma(-d2, w[r][v], p[r][v]);
            break;
        }
        if (two && test(j + 2, n[2], n[3])) break;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int y = y0 + r;
            if (r < nr && in[v]) a.p[(size_t)y * n0 + x0 + v] = p[r][v];
        }
    }
    if (first) {
        const double err = (pn > 0.0) ? num / pn : (num == 0.0 ? 0.0 : INFINITY);
        for (NewtonState* s : {a.st, a.mirror}) {
            s->m = m;
            s->fix = 0.0;
            s->t_prev = tprev;
            s->err = err;
            s->pnorm = pn;
            s->wnorm = wn;
            // (the record is not cleared before: no term of an earlier loop)
            for (int q = m + 1; q < kHist; ++q) s->hist[q] = 0.0;
            s->done = done;
        }
    }
}

struct ResidentShape {
    int vec, rows, cx, groups;
};

// The narrowest lanes that cover a row, then rows per wave; rows = 0: too
// large.
ResidentShape resident_shape(const Op& op) {
    ResidentShape g{};
    for (int vec : {1, 2}) {
        const int cx = (op.n[0] + 64 * vec - 1) / (64 * vec);
        if (cx > (vec == 1 ? 1 : kResWaves)) continue;
        // as many strips as there are waves for, of at least two rows
        const int groups = std::min(kResWaves / cx, op.n[1] / 2);
        if (groups < 1) break;
        const int rows = (op.n[1] + groups - 1) / groups;
        // (more rows would not fit the registers with edge columns or with
        // one point per lane)
        if (rows * vec > (cx > 1 || vec == 1 ? 24 : kResMaxPoints)) continue;
        g.vec = vec;
        g.cx = cx;
        g.rows = rows;
        g.groups = groups;
        break;
    }
    return g;
}

template <int V, int R, int C, bool WIDE = false>
hipError_t go(const ResidentArgs& a, hipStream_t s) {
    if (a.bc == EXPI_INTERIOR_ONLY)
        hipLaunchKernelGGL((resident2d_loop<V, R, C, WIDE, true>), dim3(1), dim3(kResWaves * 64), 0, s, a);
    else
        hipLaunchKernelGGL((resident2d_loop<V, R, C, WIDE, false>), dim3(1), dim3(kResWaves * 64), 0, s, a);
    return hipGetLastError();
}

}  // namespace

// The grid fits one workgroup's registers, in FP64 with a constant
// coefficient.
bool resident2d_supported(const Op& op, int tw, int m_max) {
    return op.kind == 0 && op.dim == 2 && op.coef == EXPI_COEF_CONST && tw == 0 && m_max <= kMaxResidentDegree &&
           op.size <= kResWaves * 64 * kResMaxPoints && resident_shape(op).rows > 0;
}

hipError_t launch_resident2d(const Op& op, ResidentArgs a, double alpha, hipStream_t s) {
    const ResidentShape g = resident_shape(op);
    for (int q = 0; q < 2; ++q) a.n[q] = op.n[q];
    a.bc = op.bc;
    a.cx = g.cx;
    a.groups = g.groups;
    a.afx = alpha * (op.c0 * (1.0 / (op.h[0] * op.h[0])));
    a.afy = alpha * (op.c0 * (1.0 / (op.h[1] * op.h[1])));
    a.afy2 = a.afy + a.afy;
    // (strips have g.rows rows or one less; at least two)
    if (g.vec == 1) {
        if (g.rows <= 4) return go<1, 4, 2>(a, s);
        if (g.rows <= 8) return go<1, 8, 4>(a, s);
        if (g.rows <= 12) return go<1, 12, 4>(a, s);
        if (g.rows <= 16) return go<1, 16, 4>(a, s);
        if (g.rows <= 24) return go<1, 24, 8>(a, s);
    } else if (g.cx > 1) {
        if (g.rows <= 4) return go<2, 4, 2, true>(a, s);
        if (g.rows <= 8) return go<2, 8, 4, true>(a, s);
        if (g.rows <= 12) return go<2, 12, 4, true>(a, s);
    } else {
        if (g.rows <= 4) return go<2, 4, 2>(a, s);
        if (g.rows <= 6) return go<2, 6, 2>(a, s);
        if (g.rows <= 8) return go<2, 8, 2>(a, s);
        if (g.rows <= 12) return go<2, 12, 4>(a, s);
        if (g.rows <= 16) return go<2, 16, 4>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace expi

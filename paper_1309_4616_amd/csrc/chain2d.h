// T consecutive Newton products per pass on 2D stencils (T steps of the
// Newton recurrence of Sec. III-C; the products are eq. (3)):
//
//   w_{j+l} = alpha A w_{j+l-1} + beta_{j+l-1} w_{j+l-1},  p += d_{j+l} w_{j+l},  l = 1..T
//
// with the norms of every w_{j+l} and p_{j+l}, so that the stop test can be
// applied at each degree afterwards.  w_j and p are read once, w_{j+T} and p
// written once: 32 B per point (FP64) for T products.
//
// What bounds it: HBM beyond the last-level cache.  At 8192^2 FP64 a pass
// of six products takes 464 to 470 us and moves 2.2 GB, a pair sweep 424, so
// phi_1 of degree 25 takes 2.3 ms against 5.5 ms in pairs.  The arithmetic is
// behind it, not far off: 25 FP64 instructions per point and product are 256
// us for six at the device's 39e12 lane operations per second, about 280 with
// what strips and tiles form twice, and the time is the same with one or two
// waves per SIMD.  A seventh level would need a seventh slot in every queue.
// On grids that fit the caches the launches count: fewer of them, and fewer
// stop tests.
//
// Layout.  A wave owns a strip of 64 V columns and marches down `march` rows.
// Level l is formed one row behind level l-1, so step s of the march brings
// in row s of w_j and forms row s-l of level l for l = 1..T; x neighbours
// come from the adjacent lanes by wave shifts, the rows above and below from
// register queues.  Strips and row tiles overlap instead of exchanging
// halos: level l is right on the strip less l columns at each inner end and
// on the tile less (plus the T rows loaded beyond it) l rows, so HX >= T
// columns at each inner end of a strip are computed but not stored.  That
// wastes 2 HX of 64 V columns (6% at V = 2, T = 4) and 2T rows of loads per
// tile, and costs no exchange, no LDS and no barrier.
//
// The march is unrolled six rows per block and every queue is indexed by row
// modulo 6, so the queues rotate by renaming: rows s+1 to s+3 of w_j load
// straight into slots that rows s-5 to s-3 have left.  (With the rows ahead
// in registers of their own, copied into the queue when their turn came,
// the compiler moved them at the loop's end and the wave waited there for
// every load in flight: 516 us per pass at 8192^2, T = 6.)  A tile starts
// with 2T steps that only fill the levels, each from its first valid row on.
#pragma once

#include "sweep_common.h"

namespace expi {
namespace chain {

constexpr int kWaves = 4;        // waves per workgroup
constexpr int kStride = 16;      // doubles per workgroup in the partials

// V values of type T at byte offset voff (per lane) + soff (scalar).
template <class TM, class TC, int V>
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, int voff, int soff, TC (&o)[V]) {
    struct P {
        TM v[V];
    };
    constexpr int N = (int)sizeof(TM) * V;
    P p;
    if constexpr (N == 4)
        p = __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    else if constexpr (N == 8)
        p = __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    else
        p = __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
#pragma unroll
    for (int v = 0; v < V; ++v) o[v] = (TC)p.v[v];
}

// Stores of at most 8 bytes: a store of more bytes needs a wait state before
// its data registers are written again, which the compiler has been seen to
// omit.
template <class TW, int V, int AUX>
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, int voff, int soff, const TW (&o)[V]) {
    typedef unsigned U2 __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(TW) * V == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, o[0]), r, voff, soff, AUX);
    } else {
        constexpr int per = 8 / (int)sizeof(TW);
        struct P {
            TW v[per];
        };
#pragma unroll
        for (int h = 0; h < V / per; ++h) {
            P q;
#pragma unroll
            for (int e = 0; e < per; ++e) q.v[e] = o[per * h + e];
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, q), r, voff + 8 * h, soff, AUX);
        }
    }
}

constexpr int kRows = 6;         // rows per unrolled block (slots of every queue)

// Columns at an inner end of a strip that are computed but not stored: T
// rounded up to whole lanes.  Streaming stores go out as whole 128-byte
// lines, so there the strips start on lines (8 columns of doubles at each
// end).
constexpr int halo_columns(int n, int vec, bool stream) { return stream ? 8 : (n + vec - 1) / vec * vec; }

// Coefficient kinds of the kernel: constant; a position-dependent
// coefficient a (stored field, or c0 + c1 X(x) Y(y) formed row by row);
// c0 D(x, y) times the Laplacian.
enum Coef : int { C_CONST = 0, C_FIELD = 1, C_SEP = 2, C_DLAP = 3 };

// One tile: strip t0, rows [t1 march, (t1+1) march).  s: ||r||^2 (a.first),
// then ||w||^2, ||p||^2 of each product.  The formulas are those of the pair
// sweep (constant coefficient) and of the single sweep (the others), term by
// term, so FP32 results do not depend on how the products are grouped.
template <class TW, int V, int T, int COEF, bool IO, bool STREAM>
__device__ __forceinline__ void chain_tile(const ChainArgs& a, int t0, int t1, double (&s)[2 * T + 1]) {
    using TC = TW;
    constexpr int U = kRows;
    constexpr int sz = (int)sizeof(TW);
    constexpr int HX = halo_columns(T, V, STREAM);
    constexpr int OUT = 64 * V - 2 * HX;
    constexpr bool kVar = (COEF != C_CONST);
    constexpr bool kA = (COEF == C_FIELD || COEF == C_SEP);
    const int lane = threadIdx.x & 63;
    const int n0 = a.n[0], n1 = a.n[1];
    const int i = t0 * OUT + lane * V;
    const int kb = t1 * a.march, ke = min(kb + a.march, n1);
    const bool in = i < n0;
    // columns this strip stores: all but HX at an end shared with another
    const bool act = in && (t0 == 0 || lane * V >= HX) && (t0 == a.tiles0 - 1 || lane * V < 64 * V - HX);
    const int ic = in ? i : (n0 - V);
    const int nbytes = n0 * n1 * sz;
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.x), 0, nbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, nbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(a.p, 0, nbytes, 0x00020000);
    // the sum read: p, or the start vector itself when the chain opens a loop
    const __amdgpu_buffer_rsrc_t rq =
        __builtin_amdgcn_make_buffer_rsrc(a.first ? const_cast<void*>(a.x) : a.p, 0, nbytes, 0x00020000);
    const int vo = ic * sz;
    const int vp = act ? vo : nbytes;      // of p only what the tile stores
    auto clampr = [&](int k) { return min(max(k, 0), n1 - 1); };
    auto roff = [&](int k) { return n0 * clampr(k) * sz; };
    const bool dir = (a.bc == EXPI_DIRICHLET0);
    const TC alpha = (TC)a.alpha;
    const bool opens = a.first != 0;
    const TC d0 = (TC)a.d0;
    TC beta[T], d[T];
#pragma unroll
    for (int l = 0; l < T; ++l) {
        beta[l] = (TC)a.beta[l];
        d[l] = (TC)a.d[l];
    }
    // constant coefficient: x weights alpha f and alpha times the x part of
    // the diagonal, 0 beyond the row's end
    const TC afx = (TC)(a.alpha * a.c0ih[0]), afy = (TC)(a.alpha * a.c0ih[1]);
    TC axm[V], axq[V], adx[V];
    bool xb[V];
    // other coefficients: existence of the x neighbours
    bool exm[V], exq[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int x = i + v;
        exm[v] = x > 0;
        exq[v] = x < n0 - 1;
        xb[v] = IO && !(exm[v] && exq[v]);
        if constexpr (!kVar) {
            axm[v] = in && exm[v] ? afx : (TC)0;
            axq[v] = in && exq[v] ? afx : (TC)0;
            adx[v] = diag_part<TC>(afx, exm[v] || dir, exq[v] || dir);
        }
    }
    const TC ihx = (TC)a.ih2[0], ihy = (TC)a.ih2[1];
    const TC c0 = (TC)a.c0, c1 = (TC)a.c1;
    // position-dependent coefficient: rows of a, prefetched
    const __amdgpu_buffer_rsrc_t rf = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double*>(COEF == C_SEP ? a.ty : a.field), 0, COEF == C_SEP ? n1 * 8 : n0 * n1 * 8, 0x00020000);
    TC Xv[V];
    if constexpr (COEF == C_SEP) {
#pragma unroll
        for (int v = 0; v < V; ++v) Xv[v] = (TC)a.tx[ic + v];
    }
    constexpr int VA = (COEF == C_SEP) ? 1 : V;
    auto a_load = [&](int k, double (&o)[VA]) {
        if constexpr (COEF == C_SEP) bload<double, double, 1>(rf, 0, clampr(k) * 8, o);
        else if constexpr (COEF == C_FIELD) bload<double, double, V>(rf, ic * 8, n0 * clampr(k) * 8, o);
    };
    auto a_row = [&](const double (&t)[VA], TC (&o)[V]) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if constexpr (COEF == C_SEP) o[v] = c0 + c1 * ((TC)t[0] * Xv[v]);
            else o[v] = (TC)t[v];
        }
    };
    const double poff = dir ? 1.0 : (a.bc == EXPI_NEUMANN0 ? 0.5 : 0.0);
    TC dfx[V + 1];   // D-Laplacian: x face weights
    if constexpr (COEF == C_DLAP) {
#pragma unroll
        for (int v = 0; v <= V; ++v) {
            const int x = i + v;       // face between x-1 and x
            const bool e = x > 0 && x < n0;
            dfx[v] = (x > n0 || !in) ? (TC)0 : face_weight<TC>(e, dir, c0, c0) * ihx;
        }
    }

    TC W[U][V], L[T][U][V], P[U][V];
    // var: rows of a (or of the y table) as stored, and the face weights of a
    // row (left faces and the right face of the last point; the face towards
    // the row above), or D
    double A[U][VA];
    TC FX[U][V + 1], FZ[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            W[u][v] = P[u][v] = (TC)0;
            FZ[u][v] = (TC)0;
            FX[u][v] = (TC)0;
            for (int l = 0; l < T; ++l) L[l][u][v] = (TC)0;
        }
        FX[u][V] = (TC)0;
    }
    // the product of level l (1..T) on row q, from rows q-1, q, q+1 of the
    // level below (wm, wc, wq); xf, zf: face weights of row q, zq: those
    // towards row q+1
    auto product = [&](int l, int q, const TC (&wm)[V], const TC (&wc)[V], const TC (&wq)[V], const TC (&xf)[V + 1],
                       const TC (&zf)[V], const TC (&zq)[V], TC (&o)[V]) {
        const bool em = q > 0, eq = q < n1 - 1;
        const bool rb = IO && !(em && eq);
        const TC left = dpp_shift0<kDppWaveShr1>(wc[V - 1]);
        const TC right = dpp_shift0<kDppWaveShl1>(wc[0]);
        if constexpr (!kVar) {
            const TC aym = em ? afy : (TC)0;
            const TC ayq = eq ? afy : (TC)0;
            const TC cdy = minus<TC>(beta[l - 1], diag_part<TC>(afy, em || dir, eq || dir));
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const TC wl = (v > 0) ? wc[v - 1] : left;
                const TC wr = (v < V - 1) ? wc[v + 1] : right;
                TC u = const_product<TC>(axm[v], axq[v], aym, ayq, minus<TC>(cdy, adx[v]), wl, wr, wm[v], wq[v], wc[v]);
                if constexpr (IO) u = (xb[v] || rb) ? beta[l - 1] * wc[v] : u;
                o[v] = (TC)(TW)u;
            }
        } else {
            // values beyond the grid are zero in every level (loads there
            // give zero, weights beyond a row's end are zero, rows beyond the
            // grid are cleared here), which is what a missing Dirichlet
            // neighbour reads
            const bool inside = q >= 0 && q < n1;
            const TC dzm = face_weight<TC>(em, dir, c0, c0) * ihy;
            const TC dzq = face_weight<TC>(eq, dir, c0, c0) * ihy;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const TC wl = (v > 0) ? wc[v - 1] : left;
                const TC wr = (v < V - 1) ? wc[v + 1] : right;
                TC fxm, fxq, fzm, fzq;
                if constexpr (COEF == C_DLAP) {
                    fxm = dfx[v];
                    fxq = dfx[v + 1];
                    fzm = dzm;
                    fzq = dzq;
                } else {
                    fxm = xf[v];
                    fxq = xf[v + 1];
                    fzm = zf[v];
                    fzq = zq[v];
                }
                TC Aw = fxm * (wl - wc[v]) + fxq * (wr - wc[v]) + fzm * (wm[v] - wc[v]) + fzq * (wq[v] - wc[v]);
                if constexpr (COEF == C_DLAP) Aw *= zf[v];
                if constexpr (IO) Aw = (xb[v] || rb) ? (TC)0 : Aw;
                const TC u = (TC)(TW)(alpha * Aw + beta[l - 1] * wc[v]);
                o[v] = (inside && i + v < n0) ? u : (TC)0;
            }
        }
    };
    // face weights of row k from a of rows k-1 (ap) and k (ac)
    auto weights = [&](int k, const TC (&ap)[V], const TC (&ac)[V], TC (&xf)[V + 1], TC (&zf)[V]) {
        const TC al = dpp_shift0<kDppWaveShr1>(ac[V - 1]);
        const TC ar = dpp_shift0<kDppWaveShl1>(ac[0]);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const TC nb = (v > 0) ? ac[v - 1] : al;
            xf[v] = (i + v < n0) ? face_weight<TC>(exm[v], dir, ac[v], nb) * ihx : (TC)0;
            // the face between rows k-1 and k; at k = 0 that of row 0, at
            // k = n1 that of row n1 - 1 (a of the clamped row n1 is its own)
            zf[v] = face_weight<TC>(k > 0 && k < n1, dir, ac[v], ap[v]) * ihy;
        }
        // (the right face of an inner point is the left face of the next one)
        xf[V] = (i + V - 1 < n0) ? face_weight<TC>(exq[V - 1], dir, ac[V - 1], ar) * ihx : (TC)0;
    };

    // Steps r = 0, 1, ...; step r brings in row s0 + r of w_j.  The first NB
    // blocks only fill the levels: E idle steps, then 2T steps (row kb - T
    // comes in at step E), then every step puts out a row.
    constexpr int NB = (2 * T + U - 1) / U, E = NB * U - 2 * T;
    constexpr int AH = 3;            // rows loaded ahead
    const int s0 = kb - T - E;
    auto w_load = [&](int r, TC (&o)[V]) { bload<TW, TC, V>(rw, vo, roff(s0 + r), o); };
#pragma unroll
    for (int r = E; r < AH; ++r) w_load(r, W[r]);
    if constexpr (kA) {
#pragma unroll
        for (int r = E - 1; r < AH; ++r) a_load(s0 + r, A[(r + U) % U]);
    }
    // one block of U steps from step r0; BLK counts the filling blocks
    auto block = [&](auto blk, int r0) {
        constexpr int BLK = decltype(blk)::value;
        constexpr bool kOut = BLK >= NB;
#pragma unroll
        for (int st = 0; st < U; ++st) {
            const int rr = BLK * U + st;      // the step, in the filling blocks
            const int k = s0 + r0 + st;       // the row of w_j that comes in
            const int q = k - T;              // the row that goes out
            if (kOut || rr + AH >= E) w_load(r0 + st + AH, W[(st + AH) % U]);
            if constexpr (kA) {
                if (kOut || rr + AH >= E - 1) a_load(k + AH, A[(st + AH) % U]);
            }
            if (kOut || rr + AH >= NB * U) bload<TW, TC, V>(rq, vp, roff(q + AH), P[(st + AH) % U]);
            if (!kOut && rr < E) continue;
            if constexpr (kVar) {
#pragma unroll
                for (int v = 0; v < V; ++v) W[st][v] = (k >= 0 && k < n1 && i + v < n0) ? W[st][v] : (TC)0;
            }
            if constexpr (kA) {
                TC ap[V], ac[V];
                a_row(A[(st + U - 1) % U], ap);
                a_row(A[st], ac);
                weights(k, ap, ac, FX[st], FZ[st]);
            } else if constexpr (COEF == C_DLAP) {
                // D of row k
#pragma unroll
                for (int v = 0; v < V; ++v)
                    FZ[st][v] = d_coefficient<TC>((TC)((i + v + poff) * a.hpos[0]), (TC)((k + poff) * a.hpos[1]));
            }
#pragma unroll
            for (int l = 1; l <= T; ++l) {
                // level l has its first valid row 2l steps after the first row
                if (!kOut && rr - E < 2 * l) continue;
                const int r = (st - l + 2 * U) % U, rm = (r + U - 1) % U, rq_ = (r + 1) % U;
                const auto& B = (l == 1) ? W : L[l > 1 ? l - 2 : 0];
                product(l, k - l, B[rm], B[r], B[rq_], FX[r], FZ[r], FZ[rq_], L[l - 1][r]);
            }
            if constexpr (kOut) {
                const int r = (st - T + 2 * U) % U;
                const bool valid = q < ke;
                TC wo[V], po[V];
                TC pl[T + 1][V];
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    pl[0][v] = P[st][v];
                    // (written out as the single and pair sweeps round it)
                    TC pv = opens ? __builtin_elementwise_fma(d0, pl[0][v], d[0] * L[0][r][v])
                                  : __builtin_elementwise_fma(d[0], L[0][r][v], pl[0][v]);
                    pl[1][v] = pv;
#pragma unroll
                    for (int l = 1; l < T; ++l) {
                        pv = __builtin_elementwise_fma(d[l], L[l][r][v], pv);
                        pl[l + 1][v] = pv;
                    }
                    wo[v] = L[T - 1][r][v];
                    po[v] = pv;
                }
                if (act && valid) {
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        s[0] += (double)pl[0][v] * (double)pl[0][v];
#pragma unroll
                        for (int l = 0; l < T; ++l) {
                            s[2 * l + 1] += (double)L[l][r][v] * (double)L[l][r][v];
                            s[2 * l + 2] += (double)pl[l + 1][v] * (double)pl[l + 1][v];
                        }
                    }
                }
                // columns and rows that belong to other tiles are stored past
                // the buffer (dropped)
                const int vs = (act && valid) ? vo : nbytes;
                bstore<TW, V, STREAM ? 2 : 0>(ro, vs, roff(q), wo);
                bstore<TW, V, STREAM ? 2 : 0>(rp, vs, roff(q), po);
            }
        }
    };
    block(std::integral_constant<int, 0>{}, 0);
    if constexpr (NB > 1) block(std::integral_constant<int, 1>{}, U);
    static_assert(NB == 1 || NB == 2, "one or two filling blocks");
    // the first block with output stands before the loop: the waits at the
    // loop's head then count the memory operations of a previous block, not
    // those of the filling blocks, which issue fewer
    block(std::integral_constant<int, NB>{}, NB * U);
    for (int r0 = (NB + 1) * U; r0 < NB * U + (ke - kb); r0 += U) block(std::integral_constant<int, NB>{}, r0);
}

template <class TW, int V, int T, int COEF, bool IO, bool STREAM>
__global__ __launch_bounds__(kWaves * 64, 2) void chain2d_sweep(ChainArgs a) {
    if (a.guard && a.st->done != 0) return;
    double s[2 * T + 1];
#pragma unroll
    for (int q = 0; q < 2 * T + 1; ++q) s[q] = 0.0;
    const int nw = blockDim.x >> 6;
    const int G = gridDim.x * nw;
    const int w0 = __builtin_amdgcn_readfirstlane(xcd_tile(gridDim.x / kXcd) * nw + (int)(threadIdx.x >> 6));
    for (int t = w0; t < a.ntiles; t += G) chain_tile<TW, V, T, COEF, IO, STREAM>(a, t % a.tiles0, t / a.tiles0, s);
    finish_sweep_n<2 * T + 1>(a.partials, kStride, s);
}

template <class TW, int V, int T, int COEF, bool STREAM = false>
hipError_t go(int grid, const ChainArgs& a, hipStream_t s) {
    if (a.bc == EXPI_INTERIOR_ONLY)
        hipLaunchKernelGGL((chain2d_sweep<TW, V, T, COEF, true, STREAM>), dim3(grid), dim3(64 * kWaves), 0, s, a);
    else
        hipLaunchKernelGGL((chain2d_sweep<TW, V, T, COEF, false, STREAM>), dim3(grid), dim3(64 * kWaves), 0, s, a);
    return hipGetLastError();
}

}  // namespace chain
}  // namespace expi

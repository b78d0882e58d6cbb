// rd_pair.h -- register-streamed passes by pairs of wavefronts: the plain pass
// of the largest single grids.
//
// A workgroup of two wavefronts owns a strip of 64*CPL columns and a segment of
// output rows.  Both start at the middle of the segment and walk apart, one up
// and one down, each with the three-row register window per time level of
// rd_fwd_body.h.  A wavefront walking alone starts with K halo rows of every
// level; here the row before a level's first one is the partner's first row of
// that level, which the two exchange through LDS while the levels start, one
// level an iteration.  That leaves the K rows at the far end: of a 35-row walk
// a wavefront computes 1.11 times its cells instead of 1.22.
//
// What bounds it: the walk of one wavefront.  Two wavefronts a SIMD (221 VGPRs, 7
// spilled SGPRs) each issue a vector instruction every four cycles at best, 17 to
// 20 % of their time goes to waits, and the clock falls to 2.0 GHz under this load.  East and west
// neighbours come by ds_bpermute, asked for one level ahead and held there by a
// scheduling barrier: DPP operands stop two wavefronts' instructions from
// issuing side by side.  4096^2, 8 steps a pass, one GPU: 95.3 us a pass alone
// with DPP; pairs 91 with DPP, 88 with ds_bpermute, 85 with the level-0 window
// of three rows (fetched one iteration ahead) and the barrier, 75 with strips that
// end at the sides (random state; 72 on the slow-growth run's mostly quiet one).
// Three rows a
// level and K = 8 fill the registers; K = 6 at three wavefronts a SIMD took 2 %
// more per step, four wavefronts a workgroup 12 % more.
#pragma once

#include <type_traits>

#include "rd_fwd_body.h"

namespace rd {

template <int CPL>
struct PairLds {
    float row[2][2][2][CPL][64];  // wavefront, buffer, layer
};

// ROWS_IN, EDGE as in rd_fwd_body.h.  Row p of a wavefront's walk, p = 0 .. h-1,
// is its p-th row from the middle; row -1 is its partner's row 0.  Iteration
// `it` makes level-(j+1) row it-j-2 from level-j rows it-j-3, it-j-2, it-j-1.
template <class M, int CPL, int K, bool ROWS_IN, bool EDGE>
__device__ __forceinline__ void pair_body(const StreamArgsT<M> &A, const Tile<CPL> &t,
                                          PairLds<CPL> &lds)
{
    static_assert(!M::kDiag && !M::kDerived, "models of four neighbours");
    const int C = A.t.C, R = A.t.R, bc = A.t.bc;
    const unsigned pbytes = 4u * (unsigned)R * (unsigned)C;
    const unsigned rowb = 4u * (unsigned)C;
    const Buf iu(A.in, pbytes), iv(A.in + (size_t)R * C, pbytes);
    const Buf ou(A.out, pbytes), ov(A.out + (size_t)R * C, pbytes);
    const typename M::Params g = A.g;
    const int lane = (int)threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int h = (t.y1 - t.y0 + 1) / 2, mid = t.y0 + h;
    const int hs = wv ? t.y1 - mid : h;  // rows this wavefront stores
    const int d = wv ? 1 : -1, s0 = wv ? mid : mid - 1;
    const int n_real = h + K + 1;
    // Byte offset of level-0 row q - 1 of the walk.
    const unsigned off0 = (unsigned)(s0 - d) * rowb, drow = (unsigned)d * rowb;
    auto roff = [&](int q) -> unsigned {
        return ROWS_IN ? off0 + (unsigned)q * drow : row_off_near(s0 + d * (q - 1), R, C, bc);
    };
    const bool at_west = EDGE && t.cx == 0, at_east = EDGE && t.cx + CPL == C;
    const int from_left = 4 * ((lane - 1) & 63), from_right = 4 * ((lane + 1) & 63);
    auto shifted = [](int from, float x) {
        return __builtin_bit_cast(
            float, __builtin_amdgcn_ds_bpermute(from, __builtin_bit_cast(int, x)));
    };

    // Windows of levels 0 .. K-1 (slots as in rd_fwd_body.h).  The newest level-0
    // row is fetched into the oldest one's slot as soon as level 1 is made.
    float bu[K][3][CPL], bv[K][3][CPL];
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int e = 0; e < CPL; ++e) bu[j][q][e] = bv[j][q][e] = 0.0f;
    load_row<CPL, true>(iu, roff(0), t, bu[0][0]);
    load_row<CPL, true>(iv, roff(0), t, bv[0][0]);

    // S = it mod 3; all: every level is active and nothing is exchanged.
    auto iteration = [&](const int it, const int S, auto all) __attribute__((always_inline)) {
        constexpr bool kAll = decltype(all)::value;
        const int buf = it & 1;
        float tu[CPL], tv[CPL];
        struct Edges {
            float lu, ru, lv, rv;
        } edge, next;
        auto edges_of = [&](const int j) __attribute__((always_inline)) {
            const Slots sl(S, j);
            const float *uC = bu[j][sl.cs], *vC = bv[j][sl.cs];
            return Edges{shifted(from_left, uC[CPL - 1]), shifted(from_right, uC[0]),
                         shifted(from_left, vC[CPL - 1]), shifted(from_right, vC[0])};
        };
        next = edges_of(0);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const Slots sl(S, j);
            edge = next;
            if (j + 1 < K) next = edges_of(j + 1);
            __builtin_amdgcn_sched_barrier(0);
            float *uN = bu[j][sl.ps], *vN = bv[j][sl.ps];
            const float *uC = bu[j][sl.cs], *uS = bu[j][sl.ns];
            const float *vC = bv[j][sl.cs], *vS = bv[j][sl.ns];
            if (!kAll && j >= 1 && it == j + 2) {
                // the row before this level's first: the partner's first
#pragma unroll
                for (int e = 0; e < CPL; ++e) {
                    uN[e] = lds.row[1 - wv][1 - buf][0][e][lane];
                    vN[e] = lds.row[1 - wv][1 - buf][1][e][lane];
                }
            }
            float *du = j + 1 < K ? bu[j + 1][sl.cs] : tu;
            float *dv = j + 1 < K ? bv[j + 1][sl.cs] : tv;
            if (kAll || it >= j + 2) {
                if (EDGE) {
                    edge.lu = at_west ? uC[0] : edge.lu;
                    edge.lv = at_west ? vC[0] : edge.lv;
                    edge.ru = at_east ? uC[CPL - 1] : edge.ru;
                    edge.rv = at_east ? vC[CPL - 1] : edge.rv;
                }
#pragma unroll
                for (int e = 0; e < CPL; ++e) {
                    Nbhd n;
                    n.u = n.y = uC[e];
                    n.v = vC[e];
                    n.uN = uN[e];
                    n.uS = uS[e];
                    n.vN = vN[e];
                    n.vS = vS[e];
                    n.uW = e == 0 ? edge.lu : uC[e - 1];
                    n.uE = e == CPL - 1 ? edge.ru : uC[e + 1];
                    n.vW = e == 0 ? edge.lv : vC[e - 1];
                    n.vE = e == CPL - 1 ? edge.rv : vC[e + 1];
                    M::update(g, n, du[e], dv[e]);
                }
                if (!kAll && j + 1 < K && it == j + 2) {
#pragma unroll
                    for (int e = 0; e < CPL; ++e) {
                        lds.row[wv][buf][0][e][lane] = du[e];
                        lds.row[wv][buf][1][e][lane] = dv[e];
                    }
                }
            }
            if (j == 0) {
                const unsigned ro = roff(it + 1);
                load_row<CPL, true>(iu, ro, t, bu[0][(S + 1) % 3]);
                load_row<CPL, true>(iv, ro, t, bv[0][(S + 1) % 3]);
            }
        }
        const int p = it - K - 1;  // row of level K now in (tu, tv)
        if ((unsigned)p < (unsigned)hs) {
            const unsigned o = (unsigned)(s0 + d * p) * rowb;
            store_row<CPL, true>(ou, o, C, t, tu);
            store_row<CPL, true>(ov, o, C, t, tv);
        }
        // rows written in iteration it are read in it + 1, their buffer written
        // again in it + 2
        if (!kAll && it >= 2 && it <= K) lds_barrier();
    };
    constexpr int kSteady = (K + 4) / 3 * 3;  // first round with it >= K + 2
    int it = 0;
    for (; it < kSteady && it < n_real; it += 3) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (it + q >= n_real) break;
            iteration(it + q, q, std::integral_constant<bool, false>{});
        }
    }
    for (; it < n_real; it += 3) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (it + q >= n_real) break;
            iteration(it + q, q, std::integral_constant<bool, true>{});
        }
    }
}

// Tiles of A.t: every one takes vectors (pair_pass, plain_geometry).
template <class M, int CPL, int K>
__global__ __launch_bounds__(128) void pair_step_kernel(StreamArgsT<M> A)
{
    __shared__ PairLds<CPL> lds;
    Tile<CPL> t;
    if (!t.init(A.t)) return;
    // the walks name rows y0 - K - 1 .. y1 + K + 1
    const bool rows_in = t.y0 > K && t.y1 + K + 1 < A.t.R;
    if (t.edge) {
        if (rows_in)
            pair_body<M, CPL, K, true, true>(A, t, lds);
        else
            pair_body<M, CPL, K, false, true>(A, t, lds);
    } else {
        if (rows_in)
            pair_body<M, CPL, K, true, false>(A, t, lds);
        else
            pair_body<M, CPL, K, false, false>(A, t, lds);
    }
}

}  // namespace rd

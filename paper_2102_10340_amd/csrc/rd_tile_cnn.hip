// rd_tile_cnn.hip -- resident-tile passes of the Chua-Yang CNN: the tiles, halos
// and row exchange of rd_tile_body.h for a model that reads all eight neighbours
// through its output y = derive(u) and has a constant second layer.
//
// Only y has neighbours, so only y rows are kept with the columns beside them
// (those of the row above and of the row below are read too), trade places from
// step to step and go through LDS; u and the input term stay in one place per
// cell.  Per row two swizzles instead of four, half the LDS traffic.  What bounds
// a step: its ~27 vector instructions per cell, and below ~1024^2 the launches
// and barriers.  us per step, the streamed pass before in brackets: 128^2 0.55
// (1.38), 512^2 0.80 (1.81), 777x1301 1.62 (2.60), 1024^2 1.62 (2.70), 2048^2 4.0
// (5.9), 4096^2 14.9 (17.1).
#include "rd_tile.h"

namespace rd {

// y of one lane's columns of a row, and of the columns beside them.
template <int CPL>
struct OutRow {
    float y[CPL], l, r;

    __device__ __forceinline__ void edges()
    {
        l = half_from_left(y[CPL - 1]);
        r = half_from_right(y[0]);
    }
};

template <int CPL, int RW, bool SPLIT>
__device__ __forceinline__ void tile_cnn_body(const TileStepArgsT<ModelCnn> &A, int x0, int y0, int y1,
                                              char *smem)
{
    const int C = A.t.C, R = A.t.R, bc = A.t.bc, K = A.K;
    const unsigned pbytes = 4u * (unsigned)R * (unsigned)C;
    const Buf iu(A.in, pbytes), iw(A.in + (size_t)R * C, pbytes);
    const Buf ou(A.out, pbytes), ow(A.out + (size_t)R * C, pbytes);
    const CnnParams g = A.g;
    const int W = (int)blockDim.y;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int half = (int)threadIdx.x >> 5;
    HalfTile<CPL, SPLIT> t;
    t.setup(A.t, x0);
    const int q0 = 2 * wave * RW;
    const int ra = y0 - K + q0, rb = ra + RW;  // first grid row of the two blocks
    const int H = y1 - y0 + 2 * K;
    const int rlast = y1 + K - 1;  // rows past it repeat it
    // y rows in slots 1..RW before an even step, 0..RW-1 before an odd one
    float u[RW][CPL], w[RW][CPL];
    OutRow<CPL> y[RW + 1];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const unsigned r0 = row_off(min(ra + i, rlast), R, C, bc);
        const unsigned r1 = row_off(min(rb + i, rlast), R, C, bc);
        const unsigned ro = half ? r1 : r0;
        t.load(iu, ro, u[i]);
        t.load(iw, ro, w[i]);
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        if (t.any_rev) {
            t.unmirror(u[i]);
            t.unmirror(w[i]);
        }
#pragma unroll
        for (int e = 0; e < CPL; ++e) y[i + 1].y[e] = ModelCnn::derive(u[i][e]);
        y[i + 1].edges();
    }
    const int b = 2 * wave + half;
    const BlockLds<CPL> lds(smem, W, b, max(b - 1, 0), min(b + 1, 2 * W - 1));
    auto put = [&](int buf, int side, const OutRow<CPL> &r) __attribute__((always_inline)) {
        vecf<CPL> a;
#pragma unroll
        for (int e = 0; e < CPL; ++e) a[e] = r.y[e];
        lds.own[buf * lds.plane + side * 32] = a;
    };
    auto get = [&](int buf, const vecf<CPL> *p) __attribute__((always_inline)) {
        OutRow<CPL> r;
        const vecf<CPL> a = p[buf * lds.plane];
#pragma unroll
        for (int e = 0; e < CPL; ++e) r.y[e] = a[e];
        r.edges();
        return r;
    };
    // row i's step from the y rows above, at and below it; its new y row into D,
    // which may be one of them
    auto update = [&](int i, const OutRow<CPL> &N, const OutRow<CPL> &Y, const OutRow<CPL> &S,
                      OutRow<CPL> &D) __attribute__((always_inline)) {
        OutRow<CPL> o;
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
            Nbhd n;
            n.u = u[i][e];
            n.v = w[i][e];
            n.y = Y.y[e];
            n.uN = N.y[e];
            n.uS = S.y[e];
            n.uNW = e == 0 ? N.l : N.y[e - 1];
            n.uW = e == 0 ? Y.l : Y.y[e - 1];
            n.uSW = e == 0 ? S.l : S.y[e - 1];
            n.uNE = e == CPL - 1 ? N.r : N.y[e + 1];
            n.uE = e == CPL - 1 ? Y.r : Y.y[e + 1];
            n.uSE = e == CPL - 1 ? S.r : S.y[e + 1];
            float v;
            ModelCnn::update(g, n, u[i][e], v);
            o.y[e] = ModelCnn::derive(u[i][e]);
        }
        o.edges();
        D = o;
    };
    put(0, 0, y[1]);
    put(0, 1, y[RW]);
    lds_barrier();
    auto active = [&](int s) { return q0 + 2 * RW > s + 1 && q0 < H - s - 1; };
    auto even_step = [&](int s) __attribute__((always_inline)) {
        if (active(s)) {
            const OutRow<CPL> nN = get(0, lds.above), nS = get(0, lds.below);
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                update(i, i == 0 ? nN : y[i], y[i + 1],
                       i == RW - 1 ? nS : y[i + 2 > RW ? RW : i + 2], y[i]);
                if (i == 0) put(1, 0, y[0]);
                if (i == RW - 1) put(1, 1, y[RW - 1]);
            }
        }
        lds_barrier();
    };
    auto odd_step = [&](int s) __attribute__((always_inline)) {
        if (active(s)) {
            const OutRow<CPL> nS = get(1, lds.below), nN = get(1, lds.above);
#pragma unroll
            for (int i = RW - 1; i >= 0; --i) {
                update(i, i == 0 ? nN : y[i < 1 ? 0 : i - 1], y[i], i == RW - 1 ? nS : y[i + 1],
                       y[i + 1]);
                if (i == RW - 1) put(0, 1, y[RW]);
                if (i == 0) put(0, 0, y[1]);
            }
        }
        lds_barrier();
    };
    for (int s = 0; s + 2 <= K; s += 2) {
        even_step(s);
        odd_step(s + 1);
    }
    if (K & 1) even_step(K - 1);
    if (!t.lane_out) return;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int r = (half ? rb : ra) + i;
        if (r >= y0 && r < y1) {
            const unsigned ro = 4u * (unsigned)r * (unsigned)C;
            t.store(ou, ro, C, u[i]);
            t.store(ow, ro, C, w[i]);
        }
    }
}

template <int CPL, int RW>
__global__ __launch_bounds__(1024) void tile_cnn_kernel(TileStepArgsT<ModelCnn> A)
{
    extern __shared__ __align__(16) char tile_smem[];
    const int tl = xcd_tile(blockIdx.x, A.t.per_xcd);
    if (tl >= A.t.ntiles) return;
    const int strip = tl / A.t.nsegs, seg = tl - strip * A.t.nsegs;
    const int x0 = strip * A.t.wout - A.t.kpad, y0 = seg * A.t.h, y1 = min(y0 + A.t.h, A.t.R);
    if (may_split<CPL>(A.t, x0))
        tile_cnn_body<CPL, RW, true>(A, x0, y0, y1, tile_smem);
    else
        tile_cnn_body<CPL, RW, false>(A, x0, y0, y1, tile_smem);
}

TileFn<ModelCnn> tile_fn_cnn(int cpl, int rw)
{
    if (cpl == 2) {
        switch (rw) {
            case 1: return &tile_cnn_kernel<2, 1>;
            case 2: return &tile_cnn_kernel<2, 2>;
            case 3: return &tile_cnn_kernel<2, 3>;
            case 4: return &tile_cnn_kernel<2, 4>;
            case 5: return &tile_cnn_kernel<2, 5>;
            case 6: return &tile_cnn_kernel<2, 6>;
        }
    } else if (cpl == 4) {
        switch (rw) {
            case 2: return &tile_cnn_kernel<4, 2>;
            case 3: return &tile_cnn_kernel<4, 3>;
            case 4: return &tile_cnn_kernel<4, 4>;
            case 5: return &tile_cnn_kernel<4, 5>;
            case 6: return &tile_cnn_kernel<4, 6>;
        }
    }
    return nullptr;
}

}  // namespace rd

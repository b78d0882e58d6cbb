// rd_tile_adj.h -- the paired reverse passes on resident tiles.
//
// The reverse steps of rd_adj_body.h's paired passes (the same formulas, so the
// same bits for (lam, mu)) in the resident tile's layout (rd_tile_body.h): a
// workgroup keeps a tile of (lam, mu) in registers for K (even) steps; per pair
// of steps each block reads its rows of the even state E, and the row above and
// below, straight from the trajectory (fetched one pair ahead, two register sets
// in turn), rebuilds the odd state from them with the forward update, steps back
// with it, exchanges rows through LDS, and steps back with E.  Output cells add
// their products to eight float32 sums per lane, folded into double after every
// pair; each wavefront adds its total to a slot of its own, so the sums have a
// fixed order.
//
// What bounds it: at two wavefronts per SIMD (4 columns x 4 rows take all 256 VGPRs
// and spill 14, with the lam-weighted sums 22: 60 and 92 bytes a lane) the latency of
// a step, then the reads of E.  A workgroup of 8 such wavefronts fills a compute unit.
// us per reverse step on grids that the streamed pairs walk at 2.17 / 2.27 / 2.59 /
// 3.95: 128^2 1.08, 256^2 1.11, 512^2 1.56, 1024^2 2.81.
#pragma once
#include "rd_adj_body.h"
#include "rd_tile_body.h"

namespace rd {

struct TileAdjArgs {
    TileArgs t;
    const float *in_l, *in_m;
    float *out_l, *out_m;
    const float *states;    // the K/2 even states the pass reads, oldest first
    unsigned state_stride;  // bytes from one to the next
    Gene g;
    int K;                  // reverse steps of the pass (even)
    double *partial;        // [>= ntiles * wavefronts][NSUM], accumulated
};

template <int CPL, int RW, bool SPLIT, bool LAMS>
__device__ __forceinline__ void tile_adjoint_body(const TileAdjArgs &A, int tile, int x0, int y0, int y1,
                                                  char *smem)
{
    const int C = A.t.C, R = A.t.R, bc = A.t.bc, K = A.K, P = K / 2;
    const unsigned pbytes = 4u * (unsigned)R * (unsigned)C;
    const Buf il(A.in_l, pbytes), im(A.in_m, pbytes);
    const Buf ol(A.out_l, pbytes), om(A.out_m, pbytes);
    const Buf sb(A.states, (unsigned)(P - 1) * A.state_stride + 2u * pbytes);
    const Gene g = A.g;
    const AdjConst kc(g);
    const int W = (int)blockDim.y;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int lane = (int)threadIdx.x, half = lane >> 5;
    HalfTile<CPL, SPLIT> t;
    t.setup(A.t, x0);
    const int q0 = 2 * w * RW;
    const int ra = y0 - K + q0, rb = ra + RW;
    const int H = y1 - y0 + 2 * K, rlast = y1 + K;
    unsigned ro[RW + 2];  // byte offsets of rows -1 .. RW of the lane's block
#pragma unroll
    for (int i = 0; i < RW + 2; ++i) {
        const unsigned r0 = row_off(min(ra + i - 1, rlast), R, C, bc);
        const unsigned r1 = row_off(min(rb + i - 1, rlast), R, C, bc);
        ro[i] = half ? r1 : r0;
    }
    Row<CPL> x[RW + 1];               // (lam, mu), slots as in the forward tile
    Row<CPL> ea[RW + 2], eb[RW + 2];  // even states, rows -1 .. RW
    // the E rows of pair p
    auto fetch = [&](int p, Row<CPL> (&e)[RW + 2]) __attribute__((always_inline)) {
        if (p < P) {
            const unsigned so = (unsigned)(P - 1 - p) * A.state_stride;
#pragma unroll
            for (int i = 0; i < RW + 2; ++i) {
                t.load(sb, ro[i], e[i].u, so);
                t.load(sb, ro[i], e[i].v, so + pbytes);
            }
        }
    };
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        t.load(il, ro[i + 1], x[i + 1].u);
        t.load(im, ro[i + 1], x[i + 1].v);
    }
    fetch(0, ea);
    if (t.any_rev) {
#pragma unroll
        for (int i = 1; i <= RW; ++i) {
            t.unmirror(x[i].u);
            t.unmirror(x[i].v);
        }
    }
    const int b = 2 * w + half;
    const BlockLds<CPL> lds(smem, W, b, max(b - 1, 0), min(b + 1, 2 * W - 1));
    Edge E[RW];
    lds.put(0, 0, x[1]);
    lds.put(0, 1, x[RW]);
#pragma unroll
    for (int i = 0; i < RW; ++i) E[i] = edge_of(x[i + 1]);
    bool cnt[RW];  // the lane's cells of row i are output cells
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int r = (half ? rb : ra) + i;
        cnt[i] = t.lane_out && r >= y0 && r < y1;
    }
    float acc[NSUM];
    double dacc[NSUM];
#pragma unroll
    for (int k = 0; k < NSUM; ++k) {
        acc[k] = 0.0f;
        dacc[k] = 0.0;
    }
    lds_barrier();
    auto active = [&](int s) { return q0 + 2 * RW > s + 1 && q0 < H - s - 1; };
    // one reverse step of row C between N and S with state row (su, sv)
    auto back = [&](const Row<CPL> &N, const Row<CPL> &Cr, const Row<CPL> &S, const Edge &e4,
                    const Row<CPL> &st, bool count, Row<CPL> &D) __attribute__((always_inline)) {
        Row<CPL> o, L;
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
            const float lW = e == 0 ? e4.lu : Cr.u[e - 1], lE = e == CPL - 1 ? e4.ru : Cr.u[e + 1];
            const float mW = e == 0 ? e4.lv : Cr.v[e - 1], mE = e == CPL - 1 ? e4.rv : Cr.v[e + 1];
            L.u[e] = __builtin_fmaf(-4.0f, Cr.u[e], (N.u[e] + S.u[e]) + (lW + lE));
            L.v[e] = __builtin_fmaf(-4.0f, Cr.v[e], (N.v[e] + S.v[e]) + (mW + mE));
            adj_cell<true, LAMS>(kc, Cr.u[e], Cr.v[e], L.u[e], L.v[e], st.u[e], st.v[e], 0, 0.0f,
                                 o.u[e], o.v[e], acc);
        }
        if (count) {  // cells outside the output may hold anything
#pragma unroll
            for (int e = 0; e < CPL; ++e)
                if (!SPLIT || t.cx + e < C) {
                    const float u = st.u[e], v = st.v[e], l = Cr.u[e], m = Cr.v[e];
                    acc[S_LLU] = __builtin_fmaf(L.u[e], u, acc[S_LLU]);
                    acc[S_LMV] = __builtin_fmaf(L.v[e], v, acc[S_LMV]);
                    if (LAMS) {
                        acc[S_LU] = __builtin_fmaf(l, u, acc[S_LU]);
                        acc[S_LU3] = __builtin_fmaf(l * u, u * u, acc[S_LU3]);
                        acc[S_LV] = __builtin_fmaf(l, v, acc[S_LV]);
                    }
                    acc[S_MU] = __builtin_fmaf(m, u, acc[S_MU]);
                    acc[S_MV] = __builtin_fmaf(m, v, acc[S_MV]);
                    acc[S_M] += m;
                }
        }
        D = o;
    };
    auto pair = [&](int p, Row<CPL> (&e)[RW + 2], Row<CPL> (&enext)[RW + 2]) __attribute__((always_inline)) {
        fetch(p + 1, enext);
        if (t.any_rev) {
#pragma unroll
            for (int i = 0; i < RW + 2; ++i) {
                t.unmirror(e[i].u);
                t.unmirror(e[i].v);
            }
        }
        if (active(2 * p)) {
            const Row<CPL> nN = lds.get(0, lds.above), nS = lds.get(0, lds.below);
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                Row<CPL> o;  // the odd state, rebuilt
                row_update<ModelFHN, CPL>(g, e[i], e[i + 1], e[i + 2], edge_of(e[i + 1]), o);
                back(i == 0 ? nN : x[i], x[i + 1], i == RW - 1 ? nS : x[i + 2 > RW ? RW : i + 2], E[i], o,
                     cnt[i], x[i]);
                if (i == 0) lds.put(1, 0, x[0]);
                if (i == RW - 1) lds.put(1, 1, x[RW - 1]);
                E[i] = edge_of(x[i]);
            }
        }
        lds_barrier();
        if (active(2 * p + 1)) {
            const Row<CPL> nS = lds.get(1, lds.below), nN = lds.get(1, lds.above);
#pragma unroll
            for (int i = RW - 1; i >= 0; --i) {
                back(i == 0 ? nN : x[i < 1 ? 0 : i - 1], x[i], i == RW - 1 ? nS : x[i + 1], E[i], e[i + 1], cnt[i],
                     x[i + 1]);
                if (i == RW - 1) lds.put(0, 1, x[RW]);
                if (i == 0) lds.put(0, 0, x[1]);
                E[i] = edge_of(x[i + 1]);
            }
        }
        lds_barrier();
#pragma unroll
        for (int k = 0; k < NSUM; ++k) {
            if (!LAMS && (k == S_LU || k == S_LU3 || k == S_LV)) continue;
            dacc[k] += (double)acc[k];
            acc[k] = 0.0f;
        }
    };
    for (int p = 0; p < P; p += 2) {
        pair(p, ea, eb);
        if (p + 1 < P) pair(p + 1, eb, ea);
    }
    if (t.lane_out) {
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int r = (half ? rb : ra) + i;
            if (r >= y0 && r < y1) {
                t.store(ol, ro[i + 1], C, x[i + 1].u);
                t.store(om, ro[i + 1], C, x[i + 1].v);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NSUM; ++k) {
        if (!LAMS && (k == S_LU || k == S_LU3 || k == S_LV)) continue;
        double s = dacc[k];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) A.partial[((size_t)tile * W + w) * NSUM + k] += s;
    }
}

template <int CPL, int RW, bool LAMS>
__global__ __launch_bounds__(512) void tile_adjoint_kernel(TileAdjArgs A)
{
    extern __shared__ __align__(16) char tile_smem[];
    const int tl = xcd_tile(blockIdx.x, A.t.per_xcd);
    if (tl >= A.t.ntiles) return;
    const int strip = tl / A.t.nsegs, seg = tl - strip * A.t.nsegs;
    const int x0 = strip * A.t.wout - A.t.kpad, y0 = seg * A.t.h, y1 = min(y0 + A.t.h, A.t.R);
    if (may_split<CPL>(A.t, x0))
        tile_adjoint_body<CPL, RW, true, LAMS>(A, tl, x0, y0, y1, tile_smem);
    else
        tile_adjoint_body<CPL, RW, false, LAMS>(A, tl, x0, y0, y1, tile_smem);
}

using TileAdjFn = void (*)(TileAdjArgs);

}  // namespace rd

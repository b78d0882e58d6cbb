// rd_tile_body.h -- resident-tile passes: K steps of a cell model on tiles held
// whole in one workgroup's registers.
//
// A workgroup of W wavefronts owns a tile of 32*CPL columns by 2*W*RW rows,
// halo included.  A wavefront holds two blocks of RW rows, one per 32-lane
// half, CPL adjacent columns per lane; block b is rows [b RW, (b+1) RW) of the
// tile.  All K steps run on the registers; between steps each block publishes
// its first and last row in LDS (two buffers in turn, one barrier per step) for
// the blocks above and below.  After s steps the outermost s rows and columns
// of the tile hold garbage, so the inner R x C part shrinks by K on each side;
// only that part is written.  The halo is read from the boundary-extended grid
// (map_index), as in the streamed kernel, so results are bit-identical to it.
//
// Why this shape.  A streamed pass on a grid of up to ~2300^2 cells is bound by
// latency: few wavefronts, each walking its rows one after another through K
// dependent levels.  Here the rows of a step are independent.  Neighbour
// columns come from ds_swizzle (rotate within 32 lanes), not from DPP: on gfx950
// two wavefronts of a SIMD issue plain float32 VALU instructions side by side
// (one per 2.3-2.9 cycles measured, against 4.1-4.3 in code that holds a DPP
// shift even once in 32 instructions), and a swizzle costs about 7.  LDS writes
// are the slow side of LDS here (78 bytes per clock against 200-250 read), which
// is why only the two outer rows of a block are written.  The largest block (4
// columns x 6 rows) takes all 128 VGPRs of its 1024-thread bound and spills 7 (24
// bytes a lane).  Measured per step,
// against the streamed kernel at its tuned shape: 128^2 0.54 us (1.17), 256^2
// 0.55 (1.23), 512^2 0.75 (1.57), 1024^2 1.39 (2.26), 2048^2 3.33 (4.2).
#pragma once

#include <type_traits>

#include "rd_models.h"
#include "rd_stream.h"

namespace rd {

template <class M>
struct TileStepArgsT {
    TileArgs t;  // h = output rows of a tile, wout / kpad as for a strip of 32*CPL columns
    const float *in;
    float *out;
    typename M::Params g;
    int K;  // steps of the pass
    // recording passes (they start at an even time): the state of even level j
    // goes to rec + (j / 2) * rec_stride bytes, level 0 only if rec_first
    float *rec;
    unsigned rec_stride;
    int rec_first;
};

// Lane i of each 32-lane half receives lane i-1's (i+1's) value of its half,
// rotating (ds_swizzle rotate mode: bit 10 the direction, bits 9:5 the count).
__device__ __forceinline__ float half_from_left(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x), 0xC420));
}
__device__ __forceinline__ float half_from_right(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x), 0xC020));
}

// One lane's columns of one row, and the columns beside them.
template <int CPL>
struct Row {
    float u[CPL], v[CPL];
};
struct Edge {
    float lu, ru, lv, rv;
};

template <int CPL>
__device__ __forceinline__ Edge edge_of(const Row<CPL> &r)
{
    return Edge{half_from_left(r.u[CPL - 1]), half_from_right(r.u[0]),
                half_from_left(r.v[CPL - 1]), half_from_right(r.v[0])};
}

// D = the model's update of row C between rows N and S (D may alias any of them).
template <class M, int CPL>
__device__ __forceinline__ void row_update(const typename M::Params &g, const Row<CPL> &N,
                                           const Row<CPL> &C, const Row<CPL> &S, const Edge &E,
                                           Row<CPL> &D)
{
    Row<CPL> o;
#pragma unroll
    for (int e = 0; e < CPL; ++e) {
        Nbhd n;
        n.u = n.y = C.u[e];
        n.v = C.v[e];
        n.uN = N.u[e];
        n.uS = S.u[e];
        n.vN = N.v[e];
        n.vS = S.v[e];
        n.uW = e == 0 ? E.lu : C.u[e - 1];
        n.uE = e == CPL - 1 ? E.ru : C.u[e + 1];
        n.vW = e == 0 ? E.lv : C.v[e - 1];
        n.vE = e == CPL - 1 ? E.rv : C.v[e + 1];
        M::update(g, n, o.u[e], o.v[e]);
    }
    D = o;
}

// Column addressing of one lane.  A lane moves its CPL columns with one vector
// access (rows need only 4-byte alignment): also at the grid's edges, where the
// boundary rule maps a lane's columns onto one run of columns, reversed (`rev`)
// where the zero-flux mirror folds them.  Only lanes whose columns a fold or a
// wrap splits (the lane across the right edge where C % CPL != 0, and lanes of
// grids narrower than a run) move each column on its own; SPLIT tiles may hold
// such lanes.  Moving every column of an edge tile on its own made 777x1301 run
// at 1.60 us per step instead of 1.37.
template <int CPL, bool SPLIT>
struct HalfTile {
    int cx;                // first column of the lane (boundary-extended)
    bool lane_out;         // the lane's columns are output columns
    bool rev, any_rev;     // this lane's columns are mirrored; some lane's may be
    bool split;            // SPLIT tiles: this lane's columns are no run
    unsigned vo, mo[CPL];  // byte offsets: of the run, of each mapped column

    __device__ __forceinline__ void setup(const TileArgs &A, int x0)
    {
        const int oc = CPL * ((int)threadIdx.x & 31);
        cx = x0 + oc;
        const int m0 = map_index(cx, A.C, A.bc), m1 = map_index(cx + CPL - 1, A.C, A.bc);
        rev = m1 < m0;
        split = false;
        if (SPLIT) {
            bool up = true, down = true;
#pragma unroll
            for (int e = 0; e < CPL; ++e) {
                const int m = map_index(cx + e, A.C, A.bc);
                up &= m == m0 + e;
                down &= m == m0 - e;
                mo[e] = 4u * (unsigned)m;
            }
            rev = down;
            split = !up && !down;
        }
        any_rev = SPLIT || (A.bc != BC_PERIODIC && (x0 < 0 || x0 + 32 * CPL > A.C));
        vo = split ? 0u : 4u * (unsigned)min(m0, m1);
        lane_out = oc >= A.kpad && oc < A.kpad + A.wout && cx < A.C;
    }

    __device__ __forceinline__ void load(const Buf &b, unsigned ro, float (&x)[CPL],
                                         unsigned soff = 0) const
    {
        if (SPLIT && split) {
#pragma unroll
            for (int e = 0; e < CPL; ++e) x[e] = buf_load1(b, mo[e] + ro, soff);
        } else {
            buf_load<CPL>(b, vo + ro, soff, x);
        }
    }

    // for output lanes: their columns inside the grid are their own, in order
    __device__ __forceinline__ void store(const Buf &b, unsigned ro, int C, const float (&x)[CPL],
                                          unsigned soff = 0) const
    {
        if (SPLIT && cx + CPL > C) {
#pragma unroll
            for (int e = 0; e < CPL; ++e)
                if (cx + e < C) buf_store1(b, 4u * (unsigned)(cx + e) + ro, soff, x[e]);
        } else {
            buf_store<CPL>(b, vo + ro, soff, x);
        }
    }

    __device__ __forceinline__ void unmirror(float (&x)[CPL]) const
    {
#pragma unroll
        for (int e = 0; e < CPL / 2; ++e) {
            const float a = x[e], b = x[CPL - 1 - e];
            x[e] = rev ? b : a;
            x[CPL - 1 - e] = rev ? a : b;
        }
    }
};

// Whether a tile whose first column is x0 may hold split lanes: not where C is a
// multiple of CPL (folds and wraps then fall between runs, as tile columns and
// kpad are multiples of CPL too), nor left of the right edge with the left halo
// inside one fold.
template <int CPL>
__device__ __forceinline__ bool may_split(const TileArgs &A, int x0)
{
    return !A.vec_ok && (x0 + 32 * CPL > A.C || -x0 > A.C);
}

// The LDS through which a lane's block trades rows with its neighbours:
// [buffer][layer][block][first, last row][32 lanes] of CPL floats.
template <int CPL>
struct BlockLds {
    using V = vecf<CPL>;
    V *own;
    const V *above, *below;  // last row of the block above, first row of the one below
    int plane;

    // block b of 2 * waves; bn, bs: the blocks above and below it
    __device__ __forceinline__ BlockLds(char *smem, int waves, int b, int bn, int bs)
    {
        V *sm = (V *)smem + ((int)threadIdx.x & 31);
        own = sm + b * 64;
        above = sm + bn * 64 + 32;
        below = sm + bs * 64;
        plane = 2 * waves * 64;
    }

    __device__ __forceinline__ void put(int buf, int side, const Row<CPL> &r) const
    {
        V a, c;
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
            a[e] = r.u[e];
            c[e] = r.v[e];
        }
        own[buf * 2 * plane + side * 32] = a;
        own[buf * 2 * plane + plane + side * 32] = c;
    }

    __device__ __forceinline__ Row<CPL> get(int buf, const V *p) const
    {
        Row<CPL> r;
        const V a = p[buf * 2 * plane], c = p[buf * 2 * plane + plane];
#pragma unroll
        for (int e = 0; e < CPL; ++e) {
            r.u[e] = a[e];
            r.v[e] = c[e];
        }
        return r;
    }
};

// LDS bytes of a workgroup: [buffer][layer][block][first, last row][32 lanes].
constexpr int tile_lds_bytes(int cpl, int w) { return 2 * 2 * (2 * w) * 2 * 32 * 4 * cpl; }

template <class M, int CPL, int RW, bool SPLIT, bool REC>
__device__ __forceinline__ void tile_body(const TileStepArgsT<M> &A, int x0, int y0, int y1, char *smem)
{
    const int C = A.t.C, R = A.t.R, bc = A.t.bc, K = A.K;
    const unsigned pbytes = 4u * (unsigned)R * (unsigned)C;
    const Buf iu(A.in, pbytes), iv(A.in + (size_t)R * C, pbytes);
    const Buf ou(A.out, pbytes), ov(A.out + (size_t)R * C, pbytes);
    const typename M::Params g = A.g;
    const int W = (int)blockDim.y;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
    const int lane = (int)threadIdx.x, half = lane >> 5;
    HalfTile<CPL, SPLIT> t;
    t.setup(A.t, x0);
    const int q0 = 2 * w * RW;                     // first tile row of the wavefront
    const int ra = y0 - K + q0, rb = ra + RW;      // first grid row of its two blocks
    const int H = y1 - y0 + 2 * K;                 // tile rows in use
    const int rlast = y1 + K - 1;                  // last one; rows past it repeat it
    // Rows live in slots 1..RW before an even step and 0..RW-1 before an odd
    // one: a step writes each new row over the slot of the row just used up, so
    // the rows shift by one slot down and back up without register copies.
    Row<CPL> x[RW + 1];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const unsigned r0 = row_off(min(ra + i, rlast), R, C, bc);
        const unsigned r1 = row_off(min(rb + i, rlast), R, C, bc);
        const unsigned ro = half ? r1 : r0;
        t.load(iu, ro, x[i + 1].u);
        t.load(iv, ro, x[i + 1].v);
    }
    if (t.any_rev) {
#pragma unroll
        for (int i = 1; i <= RW; ++i) {
            t.unmirror(x[i].u);
            t.unmirror(x[i].v);
        }
    }
    const int b = 2 * w + half;
    const BlockLds<CPL> lds(smem, W, b, max(b - 1, 0), min(b + 1, 2 * W - 1));
    // Edge columns of each row, fetched as soon as the row is made.
    Edge E[RW];
    lds.put(0, 0, x[1]);
    lds.put(0, 1, x[RW]);
#pragma unroll
    for (int i = 0; i < RW; ++i) E[i] = edge_of(x[i + 1]);
    lds_barrier();
    // Step s makes valid rows s+1 .. H-s-2; a wavefront with none of them rests.
    auto active = [&](int s) { return q0 + 2 * RW > s + 1 && q0 < H - s - 1; };
    auto even_step = [&](int s) __attribute__((always_inline)) {
        if (active(s)) {
            const Row<CPL> nN = lds.get(0, lds.above), nS = lds.get(0, lds.below);
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                row_update<M, CPL>(g, i == 0 ? nN : x[i], x[i + 1],
                                   i == RW - 1 ? nS : x[i + 2 > RW ? RW : i + 2], E[i], x[i]);
                if (i == 0) lds.put(1, 0, x[0]);
                if (i == RW - 1) lds.put(1, 1, x[RW - 1]);
                E[i] = edge_of(x[i]);
            }
        }
        lds_barrier();
    };
    auto odd_step = [&](int s) __attribute__((always_inline)) {
        if (active(s)) {
            const Row<CPL> nS = lds.get(1, lds.below), nN = lds.get(1, lds.above);
#pragma unroll
            for (int i = RW - 1; i >= 0; --i) {
                row_update<M, CPL>(g, i == 0 ? nN : x[i < 1 ? 0 : i - 1], x[i],
                                   i == RW - 1 ? nS : x[i + 1], E[i], x[i + 1]);
                if (i == RW - 1) lds.put(0, 1, x[RW]);
                if (i == 0) lds.put(0, 0, x[1]);
                E[i] = edge_of(x[i + 1]);
            }
        }
        lds_barrier();
    };
    auto store = [&](const Buf &bu, const Buf &bv, unsigned soff, auto slot0)
        __attribute__((always_inline)) {
        if (!t.lane_out) return;
        const int r0 = half ? rb : ra;
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int r = r0 + i;
            if (r >= y0 && r < y1) {
                const unsigned ro = 4u * (unsigned)r * (unsigned)C;
                t.store(bu, ro, C, x[i + decltype(slot0)::value].u, soff);
                t.store(bv, ro, C, x[i + decltype(slot0)::value].v, soff);
            }
        }
    };
    const Buf ru(REC ? A.rec : A.in, REC ? (unsigned)((K - 1) / 2) * A.rec_stride + pbytes : 0u);
    const Buf rv(REC ? A.rec + (size_t)R * C : A.in,
                 REC ? (unsigned)((K - 1) / 2) * A.rec_stride + pbytes : 0u);
    auto record = [&](int s) __attribute__((always_inline)) {
        if (REC && (s > 0 || A.rec_first))
            store(ru, rv, (unsigned)(s / 2) * A.rec_stride, std::integral_constant<int, 1>{});
    };
    for (int s = 0; s + 2 <= K; s += 2) {
        record(s);
        even_step(s);
        odd_step(s + 1);
    }
    if (K & 1) {
        record(K - 1);
        even_step(K - 1);
        store(ou, ov, 0u, std::integral_constant<int, 0>{});
    } else {
        store(ou, ov, 0u, std::integral_constant<int, 1>{});
    }
}

template <class M, int CPL, int RW, bool REC>
__global__ __launch_bounds__(1024) void tile_step_kernel(TileStepArgsT<M> A)
{
    extern __shared__ __align__(16) char tile_smem[];
    const int tl = xcd_tile(blockIdx.x, A.t.per_xcd);
    if (tl >= A.t.ntiles) return;
    const int strip = tl / A.t.nsegs, seg = tl - strip * A.t.nsegs;
    const int x0 = strip * A.t.wout - A.t.kpad, y0 = seg * A.t.h, y1 = min(y0 + A.t.h, A.t.R);
    if (may_split<CPL>(A.t, x0))
        tile_body<M, CPL, RW, true, REC>(A, x0, y0, y1, tile_smem);
    else
        tile_body<M, CPL, RW, false, REC>(A, x0, y0, y1, tile_smem);
}

template <class M>
using TileFn = void (*)(TileStepArgsT<M>);

// Instances: 2 columns per lane with blocks of 1 to 6 rows (one-row blocks only
// pay on the smallest grids), 4 with 2 to 6.
template <class M, int CPL, bool REC>
TileFn<M> pick_tile_rows(int rw)
{
    if constexpr (CPL == 2) {
        if (rw == 1) return &tile_step_kernel<M, CPL, 1, REC>;
    }
    switch (rw) {
        case 2: return &tile_step_kernel<M, CPL, 2, REC>;
        case 3: return &tile_step_kernel<M, CPL, 3, REC>;
        case 4: return &tile_step_kernel<M, CPL, 4, REC>;
        case 5: return &tile_step_kernel<M, CPL, 5, REC>;
        case 6: return &tile_step_kernel<M, CPL, 6, REC>;
        default: return nullptr;
    }
}

template <class M, bool REC>
TileFn<M> pick_tile(int cpl, int rw)
{
    return cpl == 2   ? pick_tile_rows<M, 2, REC>(rw)
           : cpl == 4 ? pick_tile_rows<M, 4, REC>(rw)
                      : nullptr;
}

}  // namespace rd

// rd_tile.hip -- choice of shape and launch of the resident-tile passes
// (rd_tile_body.h).
#include <math.h>

#include "rd_tile.h"

namespace rd {

namespace {

constexpr int kCus = 256;
constexpr int kLdsPerCu = 160 * 1024;
// VGPRs of the instances, rows per block 1 .. 6 (bounds the wavefronts of a SIMD)
constexpr int kVgpr2[7] = {0, 34, 42, 49, 57, 67, 79};
constexpr int kVgpr4[7] = {0, 0, 58, 72, 88, 108, 128};
constexpr int kWaves[] = {4, 6, 8, 10, 12, 16};

// Predicted microseconds of one K-step pass.  Fitted to 1500 timed passes on
// grids of 128^2 to 2048^2, 200x700 and 777x1301 (7 % rms); on each of them the
// shape it picks is within 1.2 % of the fastest timed one, except where C is
// odd.  The terms: launch and fill; the tile reads and the writes; then per
// step the VALU work of the workgroups that share a compute unit (never less
// than one wavefront's own issue), their LDS traffic, and the barrier.
double pass_us(int R, int C, int cpl, int rw, int w, int K, int ntiles)
{
    const int vg = ((cpl == 4 ? kVgpr4[rw] : kVgpr2[rw]) + 7) / 8 * 8;
    int wps = 512 / vg;
    if (wps > 8) wps = 8;
    int occ = wps * 4 / w;
    const int by_lds = kLdsPerCu / tile_lds_bytes(cpl, w);
    if (occ > by_lds) occ = by_lds;
    if (occ < 1) occ = 1;
    const int per = (ntiles + kCus - 1) / kCus, rounds = (per + occ - 1) / occ;
    const double conc = (double)per / rounds;
    double rest = (double)(K - 1) / (2 * rw) - 1.0;  // wavefronts past the shrinking valid rows
    if (rest < 0.0) rest = 0.0;
    const double act = (w - rest) * conc;
    const double ins = 17.0 * cpl * rw;
    double step = act / 4 * ins * 3.12;
    if (step < ins * 5.5) step = ins * 5.5;
    step += 0.63 * 4 * cpl * act + 268;
    const double mb = ((double)ntiles * (2 * w * rw) * 32 * cpl * 8 + 8.0 * R * C) * 1e-6;
    const double odd = C % cpl ? 1.2 + 0.02 * ntiles / kCus * cpl * cpl : 0.0;  // column-wise edge tiles
    return 3.57 + odd + mb / 11.0 + rounds * K * step / 2400.0;
}

struct Table {
    int R = -1, C = -1;
    TileShape best[kMaxTileDepth + 1];
    double us[kMaxTileDepth + 1];
};

// Fastest shape for each pass depth on an R x C grid.
void fill_table(Table &tb, int R, int C)
{
    tb.R = R;
    tb.C = C;
    for (int K = 1; K <= kMaxTileDepth; ++K) {
        tb.us[K] = INFINITY;
        for (int cpl = 2; cpl <= 4; cpl += 2) {
            const int kpad = (K + cpl - 1) / cpl * cpl, wout = 32 * cpl - 2 * kpad;
            const long long nstrips = ((long long)C + wout - 1) / wout;
            for (int rw = cpl / 2; rw <= 6; ++rw)
                for (int w : kWaves) {
                    const int h = 2 * w * rw - 2 * K;
                    if (h < 1) continue;
                    const long long nt = nstrips * (((long long)R + h - 1) / h);
                    if (nt > 1 << 22) continue;
                    const double us = pass_us(R, C, cpl, rw, w, K, (int)nt);
                    if (us < tb.us[K]) {
                        tb.us[K] = us;
                        tb.best[K] = TileShape{cpl, rw, w, K};
                    }
                }
        }
    }
}

}  // namespace

bool tile_plan(int R, int C, long long T, TilePlan *plan)
{
    // Up to here the resident tiles are the faster kind; above, the streamed
    // kernel's wider strips waste less on halos and hide their memory traffic
    // behind the arithmetic.
    if ((long long)R * C > kMaxTileCells || T < 1) return false;
    // the last grid size's table, per thread (a program that makes a handle per
    // call fills it once)
    static thread_local Table tb;
    if (tb.R != R || tb.C != C) fill_table(tb, R, C);
    double best = INFINITY;
    for (int K = 1; K <= kMaxTileDepth; ++K) {
        const long long n = (T + K - 1) / K;  // passes, of two depths that differ by one
        const long long lo = T / n, more = T % n;
        if (more && lo + 1 > kMaxTileDepth) continue;
        const double us = (double)(n - more) * tb.us[lo] + (more ? (double)more * tb.us[lo + 1] : 0.0);
        if (us < best) {
            best = us;
            plan->passes = n;
            plan->deeper = more;
            plan->base = tb.best[lo];
            plan->deep = tb.best[more ? lo + 1 : lo];
        }
    }
    return best < INFINITY;
}

namespace {

template <class M>
hipError_t launch_as(TileFn<M> f, const float *in, float *out, int R, int C, int bc,
                     const typename M::Params &p, const TileShape &sh, hipStream_t s)
{
    const int kpad = (sh.K + sh.cpl - 1) / sh.cpl * sh.cpl;
    TileStepArgsT<M> a;
    a.t.R = R;
    a.t.C = C;
    a.t.bc = bc;
    a.t.kpad = kpad;
    a.t.wout = 32 * sh.cpl - 2 * kpad;
    a.t.h = tile_out_rows(sh);
    if (!f || a.t.wout < 1 || a.t.h < 1 || sh.K < 1 || sh.w < 1 || sh.w > 16)
        return hipErrorInvalidValue;
    if (a.t.h > R) a.t.h = R;
    a.t.nsegs = (R + a.t.h - 1) / a.t.h;
    const long long nt = ((long long)C + a.t.wout - 1) / a.t.wout * a.t.nsegs;
    if (nt > 1 << 28) return hipErrorInvalidValue;
    a.t.ntiles = (int)nt;
    a.t.per_xcd = (a.t.ntiles + 7) / 8;
    a.t.vec_ok = C % sh.cpl == 0;
    a.in = in;
    a.out = out;
    a.g = p;
    a.K = sh.K;
    const int lds = tile_lds_bytes(sh.cpl, sh.w);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)f,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(f, dim3((unsigned)(8 * a.t.per_xcd)), dim3(64, (unsigned)sh.w), lds, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_tile(const float *in, float *out, int R, int C, int bc, const Gene &g,
                       const TileShape &shape, hipStream_t s)
{
    return launch_as<ModelFHN>(tile_fn_fhn(shape.cpl, shape.rw), in, out, R, C, bc, g, shape, s);
}

hipError_t launch_tile_gs(const float *in, float *out, int R, int C, int bc, const float *params,
                          const TileShape &shape, hipStream_t s)
{
    const GrayScottParams p{params[0], params[1], params[2], params[3], params[4]};
    return launch_as<ModelGrayScott>(tile_fn_gs(shape.cpl, shape.rw), in, out, R, C, bc, p, shape, s);
}

}  // namespace rd

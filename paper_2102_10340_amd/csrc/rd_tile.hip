// rd_tile.hip -- choice of shape and launch of the resident-tile passes
// (rd_tile_body.h).
#include <math.h>

#include "rd_tile.h"

namespace rd {

namespace {

constexpr int kCus = 256;
constexpr int kLdsPerCu = 160 * 1024;
// VGPRs of the instances, rows per block 1 .. 6 (bounds the wavefronts of a SIMD)
constexpr int kVgpr2[7] = {0, 34, 43, 50, 58, 69, 81};
constexpr int kVgpr4[7] = {0, 0, 59, 72, 89, 111, 128};
constexpr int kWaves[] = {4, 6, 8, 10, 12, 16};

// Predicted microseconds of one K-step pass.  Fitted to timed passes of 128^2 to
// 2048^2, 200x700 and 777x1301, on each of which the shape it picks is within 1.2 %
// of the fastest timed one.  It ranks shapes and depths, no more: of 1248 passes timed
// since on 39 sizes it predicts 0.97 of the time at 16 steps, 0.94 at 12, 0.90 at 8,
// 0.83 at 4 and 0.75 at one (medians).  The terms: launch and
// fill; the tile reads and the writes; then per step the VALU work of the
// workgroups that share a compute unit (never less than one wavefront's own
// issue), their LDS traffic, and the barrier.
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
    return 3.57 + mb / 11.0 + rounds * K * step / 2400.0;
}

// The same for a paired reverse pass, fitted to 280 timed passes on 128^2 to
// 1500^2 (7 % rms; the picked shape within 2 % of the fastest timed one).
double adj_pass_us(int R, int C, int cpl, int rw, int w, int K, int ntiles)
{
    constexpr int kVgpr[2][5] = {{0, 0, 112, 136, 162}, {0, 0, 179, 221, 256}};
    const int vg = (kVgpr[cpl == 4][rw] + 7) / 8 * 8;
    int occ = 512 / vg * 4 / w;
    if (occ < 1) occ = 1;
    const int per = (ntiles + kCus - 1) / kCus, rounds = (per + occ - 1) / occ;
    const double conc = (double)per / rounds;
    double rest = (double)(K - 1) / (2 * rw) - 1.0;
    if (rest < 0.0) rest = 0.0;
    const double act = (w - rest) * conc;
    const double ins = 31.0 * cpl * rw;
    double step = act / 4 * ins * 1.87;
    if (step < ins * 4.76) step = ins * 4.76;
    step += 1.09 * 4 * cpl * act + 1455;
    const double mb = ((double)ntiles * (2 * w * rw) * 32 * cpl * 8 + 8.0 * R * C) * 1e-6;
    return 2.93 + mb / 3.42 + rounds * K * step / 2400.0;
}

// Output columns of a tile, and tiles of an R x C grid (0: the shape has no output).
int tile_out_cols(const TileShape &s)
{
    return 32 * s.cpl - 2 * ((s.K + s.cpl - 1) / s.cpl * s.cpl);
}
long long tiles_of(int R, int C, const TileShape &s)
{
    const int h = tile_out_rows(s), wout = tile_out_cols(s);
    if (h < 1 || wout < 1) return 0;
    return ((long long)C + wout - 1) / wout * (((long long)R + h - 1) / h);
}

// Fastest shapes of the passes on one grid size (adj: of the reverse passes, whose
// depths are even), each depth's found when it is first asked for: 1.1 us of host
// time a depth (all 16: 17 us), which a 10-step run of 128^2 in 9.6 us would pay
// for depths it cannot use.
struct Table {
    int R = 0, C = 0;
    bool adj = false;
    unsigned known = 0;  // bit K: depth K is filled in
    TileShape best[kMaxTileDepth + 1];
    double cost[kMaxTileDepth + 1];

    double us(int K)
    {
        if (!(known >> K & 1)) fill(K);
        return cost[K];
    }
    const TileShape &shape(int K)
    {
        us(K);
        return best[K];
    }

private:
    void fill(int K)
    {
        known |= 1u << K;
        cost[K] = INFINITY;
        best[K] = TileShape{0, 0, 0, 0};
        if (adj && ((K & 1) || K > 12)) return;
        for (int cpl = 2; cpl <= 4; cpl += 2)
            for (int rw = adj ? 2 : cpl / 2; rw <= (adj ? 4 : 6); ++rw)
                for (int w : kWaves) {
                    if (adj && w > 8) break;
                    const TileShape sh{cpl, rw, w, K};
                    const long long nt = tiles_of(R, C, sh);
                    if (nt < 1 || nt > 1 << 22) continue;
                    const double t = (adj ? adj_pass_us : pass_us)(R, C, cpl, rw, w, K, (int)nt);
                    if (t < cost[K]) {
                        cost[K] = t;
                        best[K] = sh;
                    }
                }
    }
};

// The tables of a thread's last kTables sizes (20 KB): a program that makes a handle
// per call finds its size again, and one that steps several live grids in turn finds
// each of theirs.  10 steps and a read of 128^2 and of 256^2 in turn: 32.6 us with
// one size kept, 19.0 with these (31.3 on the streamed kernel).
constexpr int kTables = 48;
Table &table(int R, int C, bool adj)
{
    static thread_local Table tb[kTables];
    static thread_local int last = 0, next = 0;
    if (tb[last].R == R && tb[last].C == C && tb[last].adj == adj) return tb[last];
    for (last = 0; last < kTables; ++last)
        if (tb[last].R == R && tb[last].C == C && tb[last].adj == adj) return tb[last];
    last = next;
    next = (next + 1) % kTables;
    tb[last].R = R;
    tb[last].C = C;
    tb[last].adj = adj;
    tb[last].known = 0;
    return tb[last];
}

// No pass is predicted to take less (pass_us, adj_pass_us): plans of more passes
// than the best one's time holds need not be looked at.
constexpr double kLeastPassUs = 2.9;

// The even depth of the passes through S steps with the least total time: of
// each number of passes, equally deep ones.
int even_depth(Table &tb, long long S)
{
    int best = 2;
    double least = INFINITY;
    for (int K = kMaxTileDepth; K >= 2; K -= 2) {
        const long long n = (S + K - 1) / K;
        if ((double)n * kLeastPassUs > least) break;
        int d = (int)((S + n - 1) / n);
        d += d & 1;
        const int last = (int)(S - (n - 1) * d);  // > 0: d <= K
        const double us = (double)(n - 1) * tb.us(d) + tb.us(last + (last & 1));
        if (us <= least) {
            least = us;
            best = d;
        }
    }
    return best;
}

}  // namespace

namespace {

// Whether a grid fills its tiles: one a few cells wide spends them on columns (or
// rows) folded into the halo, unless it is small enough to be bound by launches.
// Slow-down on a run of 8 steps against the streamed kernel: 4x500000 1.26, 2x1000000
// 1.39, 1x3000000 1.35, 3000000x1 1.49, 100000x3 1.35, 100000x40 (a torus) 1.22; speed-up:
// 10000x64 1.40, 100x20000 1.30, 10000x33 1.46.
bool fills_tiles(int R, int C)
{
    const long long n = (long long)R * C;
    const int m = R < C ? R : C;
    return m >= 64 || (m >= 16 && n <= 1 << 19) || n <= 1 << 16;
}

// Streamed passes that T steps take: of up to 8 each, the other models' of 1, 2, 4 or 8.
long long streamed_passes(int model, long long T)
{
    return T / 8 + (model == MODEL_FHN ? T % 8 != 0 : __builtin_popcount((unsigned)(T % 8)));
}

// Whether a T-step run of plain passes is faster on resident tiles by this plan.
// From 9000 timed passes on 60 sizes; speed-up over the streamed passes in brackets.
// Few steps are bound by memory, which a tile does not touch while it computes:
// 777x1301 3 steps (0.94), 1792^2 2 (0.79), 2048^2 4 (0.90).  Five gain 1.0 to 1.2 up to 4M
// cells, unless a compute unit has one tile of 10 wavefronts with 5 or 6 rows a lane to
// wait for (2000x600 0.94); six gain from 1.0 (2048^2) to 1.2.  The other models take two
// streamed passes for 3 and 5 (3 steps, Gray-Scott: 256^2 1.9, 1536^2 1.5), and four of the
// CNN gain 0.97 to 1.13.
// From 4.3M cells on the streamed passes fill the chip, and one pass of tiles pays for
// two of up to 10 steps (12 on a zero-flux grid) and for three: 2304^2 9 steps 1.13, 1.29
// zero-flux; 2448^2 10 1.03, 1.10, 12 1.07 zero-flux; 2400^2 11 0.93, but Gray-Scott,
// three, 1.28; the CNN 2600x2665 5 1.28, 4096^2 3 1.27, 5 1.36, 7 1.19.  Other runs gain in
// deep tiles only: 2300x2301 8 steps a pass (0.86), 9 (1.27), 16 (1.07); where pairs of
// wavefronts are the other choice 2304^2 10 (1.07 zero-flux, 0.94), 2400^2 12 (0.90, 0.82),
// 16 (1.00, 0.91), 2448^2 14 (1.06, 0.98), and a compute unit's one tile of 10 wavefronts,
// three on two of its four SIMDs, 2200^2 10 (0.95).  The CNN's streamed pass has two
// columns per lane at most: 2300x2298 8 (1.00), 2448^2 8 (1.21), 3000^2 8 (1.16); 4096^2 8
// (0.98), 9 (1.16), 12 (1.16), 16 (1.03).
bool tiles_pay(int R, int C, int bc, int model, long long T, const TilePlan &plan)
{
    const long long n = (long long)R * C;
    const TileShape &sh = plan.base;
    if (n <= kMidTileCells) {
        if (model != MODEL_FHN || T >= 6) return true;
        return n <= 4000000 && !(sh.cpl == 2 && sh.rw >= 5 && sh.w == 10);
    }
    const long long others = streamed_passes(model, T);
    const long long most = model == MODEL_FHN ? 6000000 : model == MODEL_CNN ? 20000000 : 7000000;
    if (plan.passes == 1 && n <= most &&
        (others > 2 || (others == 2 && T <= (bc == BC_ZEROFLUX ? 12 : 10))))
        return true;
    if (model == MODEL_CNN) return sh.K >= (n <= 12000000 ? 8 : 9);
    if (!pair_pass(bc, R, C, kPairCpl, kPairDepth)) return n <= 6000000 && sh.K >= 9;
    if (bc == BC_PERIODIC) return n <= 4500000 && sh.K >= 12;
    return n <= 5500000 ? sh.K >= (sh.w == 10 ? 12 : 9) : n <= 6000000 && sh.K >= 13;
}

}  // namespace

bool tile_plan(int R, int C, int bc, int model, long long T, TilePlan *plan)
{
    if ((long long)R * C > 20000000 || !fills_tiles(R, C)) return false;
    if (T < (model == MODEL_FHN ? 5 : 3) || (T == 4 && model != MODEL_CNN)) return false;
    Table &tb = table(R, C, false);
    double best = INFINITY;
    for (int K = kMaxTileDepth; K >= 1; --K) {
        const long long n = (T + K - 1) / K;  // passes, of two depths that differ by one
        if ((double)n * kLeastPassUs > best) break;
        const long long lo = T / n, more = T % n;
        if (more && lo + 1 > kMaxTileDepth) continue;
        const double us =
            (double)(n - more) * tb.us((int)lo) + (more ? (double)more * tb.us((int)lo + 1) : 0.0);
        if (us <= best) {
            best = us;
            plan->passes = n;
            plan->deeper = more;
            plan->base = tb.shape((int)lo);
            plan->deep = tb.shape((int)(more ? lo + 1 : lo));
        }
    }
    return best < INFINITY && tiles_pay(R, C, bc, model, T, *plan);
}

int tile_record_depth(int R, int C, long long n)
{
    // Speed-up of a run over the streamed recording: 8 steps 1.2 to 1.7 on 20 sizes of
    // 256^2 to 2400^2, 50 steps 1.3 to 2.1; 6 steps 1.0 to 1.35; 2 steps 0.8 to 1.0.
    // Four steps 0.99 to 1.19 on 40 sizes, but 0.93 to 1.05 where a compute unit, which
    // holds 16 wavefronts, has one tile of 8 or 10 with 5 or 6 rows a lane to wait for
    // (900x1500 0.93, 1164^2 0.94, 1201x1003 0.96; five steps of 2301x2303 0.96).
    if ((long long)R * C > (n < 6 ? 5000000 : 6000000) || !fills_tiles(R, C) || n < 4) return 0;
    const int d = even_depth(table(R, C, false), n);
    const TileShape sh = tile_shape(R, C, d);
    if (n < 6 && (d < 4 || (sh.cpl == 2 && sh.rw >= 5 && sh.w >= 8 && sh.w <= 10))) return 0;
    return d;
}

TileShape tile_shape(int R, int C, int K) { return table(R, C, false).shape(K); }

int tile_adjoint_depth(int R, int C, long long S, bool chain)
{
    // The reverse tiles pay in one round: a workgroup of more than two rows a lane fills
    // a compute unit, of two rows half of one. Speed-up over the streamed pairs: one
    // round, all gradients of 40 sizes, 1.02 to 1.5 (1024^2 50 steps, 200 tiles, 1.28;
    // 1164^2 60, 253, 1.13; 512^2, two rows, 430, 1.39), 2200x700 60 steps 0.97; beyond,
    // 2 columns 4 rows 0.63 to 0.91 (600x1000 16 steps, 399 tiles, 0.86; 1200^2 8, 950,
    // 0.66), 4 columns 0.87 to 1.01 (1400^2 24 steps, 490, 1.01). In a chain of recorded
    // segments the reverse passes share the chip with the recording of the next one, and
    // two rounds are the faster single pass (8 steps, 1400^2, 390 tiles, 1.09, 2048x1000
    // 1.11; alone 0.88, 0.91). Where columns are no multiple of 4 a lane may hold a fold
    // or a wrap and reads column by column, for which 4 columns of 4 rows have too few
    // registers (1023x1025 8 and 50 steps 0.86, 0.83, 1500x1002 0.74, 0.68). Passes of
    // two steps are bound by memory (333x1001 0.86, 1300^2 0.90); of four 512^2 1.22,
    // 1100^2 1.01.
    if (!fills_tiles(R, C) || S < 4) return 0;
    const int d = even_depth(table(R, C, true), S);
    const TileShape sh = tile_adjoint_shape(R, C, d);
    if (d < 4 || (C % 4 != 0 && sh.cpl == 4 && sh.rw == 4)) return 0;
    const bool two_rounds = sh.cpl == 2 ? sh.rw == 2 : chain && S == 8 && d == 8 && C % 4 == 0;
    return tiles_of(R, C, sh) <= (two_rounds ? 512 : 256) ? d : 0;
}

TileShape tile_adjoint_shape(int R, int C, int K) { return table(R, C, true).shape(K); }

long long tile_adjoint_slots(int R, int C, int K)
{
    const TileShape sh = tile_adjoint_shape(R, C, K);
    return tiles_of(R, C, sh) * sh.w;
}

namespace {

// The tiling of a pass; false if the shape has no output or too many tiles.
bool tile_geometry(int R, int C, int bc, const TileShape &sh, TileArgs *t)
{
    const long long nt = tiles_of(R, C, sh);
    if (sh.K < 1 || sh.w < 1 || sh.w > 16 || nt < 1 || nt > 1 << 28) return false;
    t->R = R;
    t->C = C;
    t->bc = bc;
    t->wout = tile_out_cols(sh);
    t->kpad = (32 * sh.cpl - t->wout) / 2;
    t->h = tile_out_rows(sh) < R ? tile_out_rows(sh) : R;
    t->nsegs = (R + t->h - 1) / t->h;
    t->ntiles = (int)nt;
    t->per_xcd = (t->ntiles + 7) / 8;
    t->vec_ok = C % sh.cpl == 0;
    t->anchored = 0;
    return true;
}

template <class Args>
hipError_t launch_tiles(void (*f)(Args), const Args &a, const TileShape &sh, hipStream_t s)
{
    if (!f) return hipErrorInvalidValue;
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
                       const TileShape &sh, hipStream_t s, const TileRecord *rec)
{
    TileStepArgsT<ModelFHN> a;
    if (!tile_geometry(R, C, bc, sh, &a.t)) return hipErrorInvalidValue;
    a.in = in;
    a.out = out;
    a.g = g;
    a.K = sh.K;
    a.rec = rec ? rec->at : nullptr;
    a.rec_stride = rec ? 8u * (unsigned)rec->every * (unsigned)R * (unsigned)C : 0u;
    a.rec_first = rec && rec->first;
    return launch_tiles(rec ? tile_fn_rec(sh.cpl, sh.rw) : tile_fn_fhn(sh.cpl, sh.rw), a, sh, s);
}

hipError_t launch_tile_gs(const float *in, float *out, int R, int C, int bc, const float *params,
                          const TileShape &sh, hipStream_t s)
{
    TileStepArgsT<ModelGrayScott> a;
    if (!tile_geometry(R, C, bc, sh, &a.t)) return hipErrorInvalidValue;
    a.in = in;
    a.out = out;
    a.g = GrayScottParams{params[0], params[1], params[2], params[3], params[4]};
    a.K = sh.K;
    a.rec = nullptr;
    a.rec_stride = 0;
    a.rec_first = 0;
    return launch_tiles(tile_fn_gs(sh.cpl, sh.rw), a, sh, s);
}

hipError_t launch_tile_cnn(const float *in, float *out, int R, int C, int bc, const float *params,
                           const TileShape &sh, hipStream_t s)
{
    TileStepArgsT<ModelCnn> a;
    if (!tile_geometry(R, C, bc, sh, &a.t)) return hipErrorInvalidValue;
    a.in = in;
    a.out = out;
    a.g.dt = params[0];
    for (int k = 0; k < 9; ++k) a.g.A[k] = params[1 + k];
    a.K = sh.K;
    a.rec = nullptr;
    a.rec_stride = 0;
    a.rec_first = 0;
    return launch_tiles(tile_fn_cnn(sh.cpl, sh.rw), a, sh, s);
}

hipError_t launch_tile_adjoint(const AdjPlanes &io, const float *even_states, int every,
                               long long t_top, int R, int C, int bc, const Gene &g,
                               const TileShape &sh, double *partial, bool lam_sums, hipStream_t s)
{
    TileAdjArgs a;
    if ((sh.K & 1) || (t_top & 1) || t_top < sh.K || every < 1 || sh.w > 8 ||
        !tile_geometry(R, C, bc, sh, &a.t))
        return hipErrorInvalidValue;
    a.in_l = io.in_l;
    a.in_m = io.in_m;
    a.out_l = io.out_l;
    a.out_m = io.out_m;
    a.states = even_states + (t_top - sh.K) / 2 * every * 2LL * R * C;
    a.state_stride = 8u * (unsigned)every * (unsigned)R * (unsigned)C;
    a.g = g;
    a.K = sh.K;
    a.partial = partial;
    return launch_tiles(tile_adj_fn(lam_sums, sh.cpl, sh.rw), a, sh, s);
}

}  // namespace rd

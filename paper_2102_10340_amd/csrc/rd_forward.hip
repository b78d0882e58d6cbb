// rd_forward.hip -- forward kernels of the RD-CNN step (arXiv 2102.10340,
// Sec. II.A, Eq. (1)-(3)) for gfx950.
//
//  * init_kernel        Eq. (1) first line, u = v = k_a x.
//  * naive_step_kernel  one thread per cell, one step per launch; neighbours by
//                       the boundary rule, straight from global memory.  It is
//                       the reference the blocked kernel is compared against.
//  * stream_step_kernel K steps per pass over HBM (temporal blocking).  One
//                       wavefront owns a strip of 64*CPL columns (CPL adjacent
//                       columns per lane) and a segment of H output rows; it
//                       walks down the rows once, keeping for each of the K time
//                       levels a two-row window in registers, so row r of level
//                       j+1 is made as soon as row r+1 of level j exists.  East/
//                       west neighbours across lanes come from DPP wave shifts,
//                       north/south ones from the register window; nothing goes
//                       through LDS.  The strip carries K halo columns on each
//                       side and the segment K halo rows above and below (the
//                       valid region shrinks by one cell per level), read from
//                       the boundary-extended grid (map_index), so the boundary
//                       rule costs nothing inside the loop.  Its template
//                       instances are compiled in rd_fwd_r*.hip; plain passes of
//                       8 steps, four columns per lane, go to pairs of
//                       wavefronts (rd_pair.h) where their conditions hold.
#include "rd_fwd_kernel.h"

namespace rd {

// ---------------------------------------------------------------- init

__global__ __launch_bounds__(256) void init_kernel(const float *__restrict__ x, float ka,
                                                   float *__restrict__ state, long long n)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const float u = ka * x[i];
        state[i] = u;
        state[n + i] = u;
    }
}

hipError_t launch_init(const float *x, float ka, float *state, long long n, hipStream_t s)
{
    long long blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(init_kernel, dim3((unsigned)blocks), dim3(256), 0, s, x, ka, state, n);
    return hipGetLastError();
}

// One workgroup per kInitChunk cells of one instance, found from its number by
// bisection (a batch of small grids is bound by launches: 256 of them took 2.2 us
// each plus their host time, one launch over all 10 us; with the largest instance's
// workgroups for each, one 4096^2 among 1000 of 64^2 took 3.7 ms to create, 3.2 this
// way).
__global__ __launch_bounds__(256) void batch_init_kernel(const BatchInst *__restrict__ insts,
                                                         int n, long long first,
                                                         const float *__restrict__ x, float ka,
                                                         float *__restrict__ state)
{
    const long long id = first + blockIdx.x;
    int lo = 0, hi = n;  // the last instance whose first workgroup is not past id
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (insts[mid].chunk0 <= id)
            lo = mid;
        else
            hi = mid;
    }
    const BatchInst I = insts[lo];
    const long long cells = (long long)I.R * I.C, k0 = (id - I.chunk0) * kInitChunk;
    const long long k1 = k0 + kInitChunk < cells ? k0 + kInitChunk : cells;
    const float *xi = x + I.xoff;
    float *si = state + I.off;
    for (long long k = k0 + threadIdx.x; k < k1; k += 256) {
        const float u = ka * xi[k];
        si[k] = u;
        si[cells + k] = u;
    }
}

hipError_t launch_batch_init(const BatchInst *insts, int n, long long chunks, const float *x,
                             float ka, float *state, hipStream_t s)
{
    // a launch may have fewer than 2^32 threads
    constexpr long long kMost = 1 << 23;
    for (long long first = 0; first < chunks; first += kMost) {
        const long long m = chunks - first < kMost ? chunks - first : kMost;
        hipLaunchKernelGGL(batch_init_kernel, dim3((unsigned)m), dim3(256), 0, s, insts, n, first, x,
                           ka, state);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------- finite check

__global__ __launch_bounds__(256) void fill_int_kernel(int *p, int v) { p[threadIdx.x] = v; }

// Adds the number of NaN or infinite values among x[0 .. n) to *count.  The
// count is an integer, so the order of the atomic adds does not matter.
__global__ __launch_bounds__(256) void count_nonfinite_kernel(const float *__restrict__ x,
                                                              long long n, int *count)
{
    int bad = 0;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        bad += !__builtin_isfinite(x[i]);
    if (bad) atomicAdd(count, bad);
}

hipError_t launch_count_nonfinite(const float *x, long long n, int *count, hipStream_t s)
{
    hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(1), 0, s, count, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n <= 0) return e;
    long long blocks = (n + 1023) / 1024;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(count_nonfinite_kernel, dim3((unsigned)blocks), dim3(256), 0, s, x, n, count);
    return hipGetLastError();
}

// ---------------------------------------------------------------- read

// Both planes of a state to their destinations in one launch: two copies of a
// 128^2 grid took 2 x 2.0 us of GPU time and two submissions (about 2.8 us of
// host time each), one launch 2.2 us.  vec: every pointer is 16-byte aligned and
// n a multiple of 4.
//
// Bound by memory.  Stores pass the caches by: a read's copy is not what the next
// pass reads (4096^2, a step and a read: 129 us with plain stores, 90 so, 135 with
// copies; the same up to 3100x3333).  At most kReadBlocks workgroups: after a launch
// of more than 8192 wavefronts a streamed pass, two wavefronts of which fill a SIMD,
// ran up to a third slower than after fewer (steps and a read, us, 16384 or 3072
// workgroups / 2048 / copies: 2048^2, 5 steps, 38.0 / 32.9 / 34.1; 2600x2665, 8, 76.8 /
// 63.8 / 64.3; the CNN on 4096^2, 8, 230 / 177 / 195).
constexpr int kReadBlocks = 2048;

__global__ __launch_bounds__(256) void copy_planes_kernel(const float *__restrict__ src, long long n,
                                                          float *__restrict__ u,
                                                          float *__restrict__ v, int vec)
{
    using f4 = float __attribute__((ext_vector_type(4)));
    const long long stride = (long long)gridDim.x * blockDim.x;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (vec) {
        const f4 *su = reinterpret_cast<const f4 *>(src);
        const f4 *sv = reinterpret_cast<const f4 *>(src + n);
        f4 *du = reinterpret_cast<f4 *>(u), *dv = reinterpret_cast<f4 *>(v);
        for (long long i = t; i < n / 4; i += stride) {
            const f4 a = su[i], b = sv[i];
            __builtin_nontemporal_store(a, du + i);
            __builtin_nontemporal_store(b, dv + i);
        }
    } else {
        for (long long i = t; i < n; i += stride) {
            const float a = src[i], b = src[n + i];
            __builtin_nontemporal_store(a, u + i);
            __builtin_nontemporal_store(b, v + i);
        }
    }
}

hipError_t launch_copy_planes(const float *src, long long n, float *u, float *v, hipStream_t s)
{
    const int vec = n % 4 == 0 && ((uintptr_t)src | (uintptr_t)u | (uintptr_t)v) % 16 == 0;
    long long blocks = ((vec ? n / 4 : n) + 255) / 256;
    if (blocks > kReadBlocks) blocks = kReadBlocks;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(copy_planes_kernel, dim3((unsigned)blocks), dim3(256), 0, s, src, n, u, v, vec);
    return hipGetLastError();
}

// ---------------------------------------------------------------- naive

__global__ __launch_bounds__(256) void naive_step_kernel(const float *__restrict__ in,
                                                         float *__restrict__ out, int R, int C,
                                                         int bc, Gene g)
{
    const int j = blockIdx.x * 64 + threadIdx.x;
    if (j >= C) return;
    const size_t plane = (size_t)R * C;
    const bool per = bc == BC_PERIODIC;
    const int jW = j > 0 ? j - 1 : (per ? C - 1 : j);
    const int jE = j < C - 1 ? j + 1 : (per ? 0 : j);
    for (int i = blockIdx.y * 4 + threadIdx.y; i < R; i += gridDim.y * 4) {
        const int iN = i > 0 ? i - 1 : (per ? R - 1 : i);
        const int iS = i < R - 1 ? i + 1 : (per ? 0 : i);
        const size_t k = (size_t)i * C + j;
        const float *u = in, *v = in + plane;
        float uo, vo;
        cell_update(g, u[k], v[k], u[(size_t)iN * C + j], u[(size_t)iS * C + j],
                    u[(size_t)i * C + jW], u[(size_t)i * C + jE], v[(size_t)iN * C + j],
                    v[(size_t)iS * C + j], v[(size_t)i * C + jW], v[(size_t)i * C + jE], uo, vo);
        out[k] = uo;
        out[plane + k] = vo;
    }
}

hipError_t launch_naive(const float *in, float *out, int R, int C, int bc, const Gene &g,
                        hipStream_t s)
{
    const unsigned gx = (unsigned)((C + 63) / 64);
    long long gy = ((long long)R + 3) / 4;
    if (gy > 65535) gy = 65535;
    hipLaunchKernelGGL(naive_step_kernel, dim3(gx, (unsigned)gy), dim3(64, 4), 0, s, in, out, R, C,
                       bc, g);
    return hipGetLastError();
}

// ---------------------------------------------------------------- streamed

namespace {

// The tiling from its strips: segments of h rows, h = 0 for about two resident
// wavefronts per SIMD (1024 SIMDs), `waves` wavefronts a tile.
bool cut_segments(int R, int h, int waves, StreamGeom *g)
{
    if (h <= 0) {
        long long want = 2048 / waves / g->nstrips;
        if (want < 1) want = 1;
        h = (int)(((long long)R + want - 1) / want);
        h = (h + waves - 1) / waves * waves;
        if (h < 4 * waves) h = 4 * waves;
    }
    if (h > R) h = R;
    g->h = h;
    g->nsegs = (R + h - 1) / h;
    const long long nt = (long long)g->nstrips * g->nsegs;
    if (nt > (1LL << 30)) return false;
    g->ntiles = (int)nt;
    g->per_xcd = (g->ntiles + 7) / 8;
    return true;
}

}  // namespace

bool stream_geometry(int R, int C, int cpl, int depth, int seg_rows, StreamGeom *g)
{
    if (cpl != 1 && cpl != 2 && cpl != 4) return false;
    if (depth < 1 || depth > max_depth(cpl)) return false;
    g->cpl = cpl;
    g->depth = depth;
    g->kpad = (depth + cpl - 1) / cpl * cpl;
    g->wout = 64 * cpl - 2 * g->kpad;
    if (g->wout <= 0) return false;
    g->paired = g->anchored = false;
    g->nstrips = (C + g->wout - 1) / g->wout;
    return cut_segments(R, seg_rows, 1, g);
}

bool plain_geometry(int R, int C, int bc, int cpl, int depth, int seg_rows, StreamGeom *g)
{
    if (!stream_geometry(R, C, cpl, depth, seg_rows, g)) return false;
    g->paired = pair_pass(bc, R, C, cpl, depth);
    if (!g->paired) return true;
    g->anchored = strips_anchored(bc, R, C, cpl, depth);
    if (g->anchored) g->nstrips = C > 64 * cpl ? (C - 2 * g->kpad + g->wout - 1) / g->wout : 1;
    return cut_segments(R, seg_rows > R / 2 ? R : 2 * seg_rows, 2, g);
}

namespace {

// The instance for a pass: recording mode rec (rd_fwd_body.h), cpl columns per
// lane, depth steps; null if there is none.
StreamFn pick_stream(int rec, int cpl, int depth)
{
    if (rec >= 2) {  // even-state recording: one or two columns per lane, depth <= 8
        if (cpl == 1) return rec == 2 ? stream_fn_r2c1(depth) : stream_fn_r3c1(depth);
        if (cpl == 2) return rec == 2 ? stream_fn_r2c2(depth) : stream_fn_r3c2(depth);
        return nullptr;
    }
    if (cpl == 4) return rec ? stream_fn_r1c4(depth) : stream_fn_r0c4(depth);
    if (cpl == 2) return rec ? stream_fn_r1c2(depth) : stream_fn_r0c2(depth);
    if (cpl == 1) return rec ? stream_fn_r1c1(depth) : stream_fn_r0c1(depth);
    return nullptr;
}

}  // namespace

TileArgs tile_args(int R, int C, int bc, const StreamGeom &geom)
{
    TileArgs t;
    t.R = R;
    t.C = C;
    t.bc = bc;
    t.wout = geom.wout;
    t.kpad = geom.kpad;
    t.h = geom.h;
    t.nsegs = geom.nsegs;
    t.ntiles = geom.ntiles;
    t.per_xcd = geom.per_xcd;
    t.vec_ok = (C % geom.cpl) == 0;
    t.anchored = geom.anchored;
    return t;
}

hipError_t launch_stream(const float *in, float *out, int R, int C, int bc, const Gene &g,
                         const StreamGeom &geom, hipStream_t s, float *rec, long long rec_q0,
                         bool rec_even, bool skip_level0, int rec_every)
{
    if (rec_every < 1) return hipErrorInvalidValue;
    StreamFn f = geom.paired ? (rec ? nullptr : pair_fn())
                             : pick_stream(!rec ? 0 : !rec_even ? 1 : skip_level0 ? 3 : 2, geom.cpl,
                                           geom.depth);
    if (!f) return hipErrorInvalidValue;
    StreamArgs a;
    a.t = tile_args(R, C, bc, geom);
    a.in = in;
    a.out = out;
    a.g = g;
    a.rec = rec ? rec + rec_q0 * rec_every * 2LL * R * C : nullptr;
    a.rec_stride = 8u * (unsigned)rec_every * (unsigned)R * (unsigned)C;
    hipLaunchKernelGGL(f, dim3((unsigned)(8 * geom.per_xcd)), dim3(64, geom.paired ? 2 : 1), 0, s, a);
    return hipGetLastError();
}

}  // namespace rd

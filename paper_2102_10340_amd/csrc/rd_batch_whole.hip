// rd_batch_whole.hip -- small instances of a batch held whole in one
// workgroup's registers for all steps of a run.
//
// The layout is the resident tile's (rd_tile_body.h) without a halo: a 32-lane
// half of a wavefront holds a block of RW rows, CPL adjacent columns per lane,
// and the blocks of one workgroup cover the instance exactly (R = RW * blocks,
// C = CPL * lanes).  Between steps each block publishes its first and last row
// in LDS; the edge columns come from the neighbouring lanes through LDS
// permutes.  The boundary rule sits in the addresses: a ghost row is read from
// the block at the other end (periodic) or from the block itself (zero-flux),
// and a ghost column likewise from the other end's lane or the lane's own edge
// column.  One HBM read at the start, one write at the end.
//
// What bounds it: the float32 VALU work (128x128: 272 instructions per wavefront
// and step, four wavefronts per SIMD), then the LDS writes of the outer rows.
// 256 instances of 128x128: 1.62 us per step against 4.4 us for the kernel that
// keeps the whole frame in LDS and reads three cells from it per update
// (batch_lds_kernel, which still takes the shapes this one cannot cut evenly).
#include "rd_launch.h"
#include "rd_tile_body.h"

namespace rd {

namespace {

// m ? a : b bit by bit (m all ones or all zeros per lane): v_bfi_b32
__device__ __forceinline__ float bit_select(unsigned m, float a, float b)
{
    const unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    return __builtin_bit_cast(float, (m & x) | (~m & y));
}

__device__ __forceinline__ float lane_perm(int byte_addr, float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(byte_addr, __builtin_bit_cast(int, x)));
}

// FULL: all 32 lanes of a half hold columns, so the rotating swizzle wraps at
// the grid's edge; otherwise a permute with the wrap in its addresses.
template <int CPL, int RW, bool FULL, bool PERIODIC>
__device__ __forceinline__ void whole_body(const BatchInst &I, const float *in, float *out,
                                           long long T, char *smem)
{
    const int R = I.R, C = I.C;
    const unsigned pbytes = 4u * (unsigned)R * (unsigned)C;
    const Buf iu(in + I.off, pbytes), iv(in + I.off + (size_t)R * C, pbytes);
    const Buf ou(out + I.off, pbytes), ov(out + I.off + (size_t)R * C, pbytes);
    const Gene g = I.g;
    const int lane = (int)threadIdx.x, hl = lane & 31, half = lane & 32;
    const int b = 2 * (int)threadIdx.y + (half >> 5);
    const int nb = R / RW, nl = C / CPL;  // blocks, lanes per half
    const bool mine = b < nb && hl < nl;
    const unsigned vo = mine ? 4u * ((unsigned)b * RW * (unsigned)C + (unsigned)CPL * hl) : 0u;
    const unsigned rowb = 4u * (unsigned)C;
    const unsigned mL = hl == 0 ? ~0u : 0u, mR = hl == nl - 1 ? ~0u : 0u;
    const int aL = 4 * (half + (hl == 0 ? nl - 1 : hl - 1));
    const int aR = 4 * (half + (hl >= nl - 1 ? 0 : hl + 1));
    auto edges = [&](const Row<CPL> &r) __attribute__((always_inline)) {
        Edge e;
        if (FULL)
            e = edge_of(r);
        else
            e = Edge{lane_perm(aL, r.u[CPL - 1]), lane_perm(aR, r.u[0]),
                     lane_perm(aL, r.v[CPL - 1]), lane_perm(aR, r.v[0])};
        return e;
    };
    // the ghost columns of a zero-flux grid repeat the edge column
    auto ghost = [&](const Row<CPL> &r, Edge e) __attribute__((always_inline)) {
        if (!PERIODIC) {
            e.lu = bit_select(mL, r.u[0], e.lu);
            e.lv = bit_select(mL, r.v[0], e.lv);
            e.ru = bit_select(mR, r.u[CPL - 1], e.ru);
            e.rv = bit_select(mR, r.v[CPL - 1], e.rv);
        }
        return e;
    };
    Row<CPL> x[RW + 1];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        buf_load<CPL>(iu, vo, (unsigned)i * rowb, x[i + 1].u);
        buf_load<CPL>(iv, vo, (unsigned)i * rowb, x[i + 1].v);
    }
    const int W = (int)blockDim.y;
    const BlockLds<CPL> lds(smem, W, b, b == 0 ? nb - 1 : b - 1, b >= nb - 1 ? 0 : b + 1);
    const auto *above = !PERIODIC && b == 0 ? lds.own : lds.above;
    const auto *below = !PERIODIC && b >= nb - 1 ? lds.own + 32 : lds.below;
    Edge E[RW];
    lds.put(0, 0, x[1]);
    lds.put(0, 1, x[RW]);
#pragma unroll
    for (int i = 0; i < RW; ++i) E[i] = edges(x[i + 1]);
    lds_barrier();
    // wavefronts past the last block only keep the barriers
    const bool on = 2 * __builtin_amdgcn_readfirstlane((int)threadIdx.y) < nb;
    auto even_step = [&]() __attribute__((always_inline)) {
        if (on) {
            const Row<CPL> nN = lds.get(0, above), nS = lds.get(0, below);
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                row_update<ModelFHN, CPL>(g, i == 0 ? nN : x[i], x[i + 1],
                                          i == RW - 1 ? nS : x[i + 2 > RW ? RW : i + 2],
                                          ghost(x[i + 1], E[i]), x[i]);
                if (i == 0) lds.put(1, 0, x[0]);
                if (i == RW - 1) lds.put(1, 1, x[RW - 1]);
                E[i] = edges(x[i]);
            }
        }
        lds_barrier();
    };
    auto odd_step = [&]() __attribute__((always_inline)) {
        if (on) {
            const Row<CPL> nS = lds.get(1, below), nN = lds.get(1, above);
#pragma unroll
            for (int i = RW - 1; i >= 0; --i) {
                row_update<ModelFHN, CPL>(g, i == 0 ? nN : x[i < 1 ? 0 : i - 1], x[i],
                                          i == RW - 1 ? nS : x[i + 1], ghost(x[i], E[i]), x[i + 1]);
                if (i == RW - 1) lds.put(0, 1, x[RW]);
                if (i == 0) lds.put(0, 0, x[1]);
                E[i] = edges(x[i + 1]);
            }
        }
        lds_barrier();
    };
    for (long long s = 0; s + 2 <= T; s += 2) {
        even_step();
        odd_step();
    }
    const bool odd = T & 1;
    if (odd) even_step();
    if (mine) {
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            if (odd) {
                buf_store<CPL>(ou, vo, (unsigned)i * rowb, x[i].u);
                buf_store<CPL>(ov, vo, (unsigned)i * rowb, x[i].v);
            } else {
                buf_store<CPL>(ou, vo, (unsigned)i * rowb, x[i + 1].u);
                buf_store<CPL>(ov, vo, (unsigned)i * rowb, x[i + 1].v);
            }
        }
    }
}

template <int CPL, int RW>
__device__ __forceinline__ void whole_rows(const BatchInst &I, const float *in, float *out, int bc,
                                           long long T, char *smem)
{
    const bool full = I.C == 32 * CPL;
    if (bc == BC_PERIODIC) {
        if (full)
            whole_body<CPL, RW, true, true>(I, in, out, T, smem);
        else
            whole_body<CPL, RW, false, true>(I, in, out, T, smem);
    } else {
        if (full)
            whole_body<CPL, RW, true, false>(I, in, out, T, smem);
        else
            whole_body<CPL, RW, false, false>(I, in, out, T, smem);
    }
}

template <int CPL>
__global__ __launch_bounds__(1024) void batch_whole_kernel(const BatchInst *insts,
                                                           const WholeInst *list, const float *in,
                                                           float *out, int bc, long long T)
{
    extern __shared__ __align__(16) char whole_smem[];
    const WholeInst wi = list[blockIdx.x];
    const BatchInst I = insts[wi.inst];
    switch (wi.rw) {
        case 1: whole_rows<CPL, 1>(I, in, out, bc, T, whole_smem); break;
        case 2: whole_rows<CPL, 2>(I, in, out, bc, T, whole_smem); break;
        case 3: whole_rows<CPL, 3>(I, in, out, bc, T, whole_smem); break;
        case 4: whole_rows<CPL, 4>(I, in, out, bc, T, whole_smem); break;
        case 5: whole_rows<CPL, 5>(I, in, out, bc, T, whole_smem); break;
        case 6: whole_rows<CPL, 6>(I, in, out, bc, T, whole_smem); break;
        default: break;
    }
}

}  // namespace

// The cut of an R x C instance: two columns per lane up to 64 columns, four up
// to 128, and the rows per block that divide R into at most 32 blocks, as close
// to four as there is (fewer leave more LDS writes per cell, more leave fewer
// wavefronts).  False if there is none.
bool whole_shape(int R, int C, int *cpl, int *rw)
{
    if (C % 2 == 0 && C <= 64)
        *cpl = 2;
    else if (C % 4 == 0 && C <= 128)
        *cpl = 4;
    else
        return false;
    for (int r : {4, 3, 5, 2, 6, 1})
        if (R % r == 0 && R / r <= 32) {
            *rw = r;
            return true;
        }
    return false;
}

int whole_lds_bytes(int cpl, int waves) { return tile_lds_bytes(cpl, waves); }

hipError_t launch_batch_whole(const BatchInst *insts, const WholeInst *list, int count, int cpl,
                              int waves, const float *in, float *out, int bc, long long T,
                              hipStream_t s)
{
    if (count < 1 || waves < 1 || waves > 16 || (cpl != 2 && cpl != 4)) return hipErrorInvalidValue;
    const int lds = tile_lds_bytes(cpl, waves);
    auto f = cpl == 2 ? &batch_whole_kernel<2> : &batch_whole_kernel<4>;
    const hipError_t e =
        hipFuncSetAttribute((const void *)f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(f, dim3((unsigned)count), dim3(64, (unsigned)waves), lds, s, insts, list, in,
                       out, bc, T);
    return hipGetLastError();
}

}  // namespace rd

// stencil_small_kernel: the Brillouin stencil on lattices too small to fill the chip with 64-site
// tiles (8^4 is 64 of them for 256 CUs).  What counts there is the number of dependent rounds of loads
// a wave goes through, so the work is spread as wide as it goes: a block owns 16 consecutive sites of
// one right-hand side, a wave holds them four times over, and each of the 4 * NW groups of 16 lanes takes
// its own stored slabs (40 / 32 = one or two per group with NW = 8 waves).  The slab index, and with it
// the neighbours and spin weights, then differ between the groups of a wave, so the weights sit in
// vector registers and a gamma term is applied to the lanes whose weight is not zero.  All 42 loads of a
// slab (both terms) are requested before the first is used; FP64 takes 254 VGPRs for it, two waves per
// SIMD, no spills.  The partial sums of all groups meet in LDS; thread c * 16 + l finishes component c of
// site l.  Bound by that latency, two turns of it with eight waves, three with four: 8^4 FP64 10.6 us
// (25.2 MB: 2.4 TB/s; 15.3 with every gamma term on every lane) against 21.6 with twelve waves on 64-site
// tiles, FP32 6.9 against 16.7 us.
#pragma once

#include "stencil_core.hpp"

namespace bri {

constexpr int SMALL_SITES = 16;

// v 2^e for v and v 2^e normal numbers (one integer add on the exponent)
__device__ __forceinline__ float scale_pow2(float v, int e) { return __int_as_float(__float_as_int(v) + (e << 23)); }
__device__ __forceinline__ double scale_pow2(double v, int e) {
    return __hiloint2double(__double2hiint(v) + (e << 20), __double2loint(v));
}

// the twelve components of ps at site ys
template <typename C>
__device__ __forceinline__ void load_spinor(C (&p)[4][3], const C *__restrict__ ps, unsigned ys, unsigned V) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int b = 0; b < 3; ++b) p[s][b] = ps[(size_t)(s * 3 + b) * V + ys];
}

template <class LS, int NW, bool DAG, int MODE>
__global__ __launch_bounds__(64 * NW) void stencil_small_kernel(StencilArgs a) {
    using R = typename LS::R;
    using C = typename Cx<R>::T;
    constexpr int GROUPS = 4 * NW;
    extern __shared__ __align__(16) unsigned char small_lds[];
    C(*red)[12][SMALL_SITES] = (C(*)[12][SMALL_SITES])small_lds;  // [GROUPS]
    int blk, col;
    tile_and_group(a.nslots, a.xcd_remap, blk, col);
    if (col >= a.ncol || col_done<MODE>(a, col)) return;

    const unsigned V = (unsigned)a.g.V;
    const int tid = threadIdx.x, l = tid & 15, grp = tid >> 4;
    const unsigned x = (unsigned)blk * SMALL_SITES + l;
    unsigned om[4], o0[4], op[4];
    {
        unsigned rest = x, stride = 1;
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            const unsigned Lm = (unsigned)a.g.L[mu], c = rest % Lm;
            rest /= Lm;
            om[mu] = (c == 0 ? Lm - 1 : c - 1) * stride;
            o0[mu] = c * stride;
            op[mu] = (c == Lm - 1 ? 0 : c + 1) * stride;
            stride *= Lm;
        }
    }
    const C *__restrict__ in = (const C *)a.in + (size_t)col * 12 * V;
    const typename LS::store_t *__restrict__ W = (const typename LS::store_t *)a.W;

    C acc[4][3];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int b = 0; b < 3; ++b) acc[s][b] = cmake<C>((R)0, (R)0);
    for (int j = grp; j < 40; j += GROUPS) {
        const int d0 = j % 3 - 1, d1 = (j / 3) % 3 - 1, d2 = (j / 9) % 3 - 1, d3 = j / 27 - 1;
        const unsigned y = neighbour(j, +1, om, o0, op), z = neighbour(j, -1, om, o0, op);
        const typename LS::store_t *__restrict__ Wj = W + (size_t)j * 9 * V;
        // both terms' links and spinors are requested before either is used
        C wo[3][3], wp[3][3], po[4][3], pp[4][3], chi[4][3];
        load_link<LS>(wo, Wj, x, V);
        load_spinor(po, in, y, V);
        load_link<LS>(wp, Wj, z, V);
        load_spinor(pp, in, z, V);
        const int h = (d0 != 0) + (d1 != 0) + (d2 != 0) + (d3 != 0);
        const R aw = scale_pow2((R)-0.125, -h), cw = scale_pow2((R)((DAG ? -16.0 : 16.0) / 27.0), -2 * h);
        const R c0 = cw * (R)d0, c1 = cw * (R)d1, c2 = cw * (R)d2, c3 = cw * (R)d3;
        transport_vals<C, R, false>(chi, wo, po);
        spin_accumulate(acc, chi, aw, c0, c1, c2, c3);
        transport_vals<C, R, true>(chi, wp, pp);
        spin_accumulate(acc, chi, aw, -c0, -c1, -c2, -c3);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int b = 0; b < 3; ++b) red[grp][s * 3 + b][l] = acc[s][b];
    const double alpha = block_alpha<MODE>(a, col);
    __syncthreads();

    double n0 = 0.0, n1 = 0.0;
    if (tid < 12 * SMALL_SITES) {
        const int comp = tid >> 4;
        C v = in[(size_t)comp * V + x];
        v = cmake<C>((R)a.diag * v.x, (R)a.diag * v.y);
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const C u = red[g][comp][l];
            v.x += u.x;
            v.y += u.y;
        }
        if (a.g.csw != 0.0) clover_row<LS>(v, W + (size_t)LINK_SLAB_ENTRIES * V, in, comp, x, V);
        epilogue<MODE, C, R>(a, col, comp, x, V, v, n0, n1, alpha);
    }
    if constexpr (MODE == EPI_NORMS || MODE == EPI_CG_R) {
        // the twelve components sit in the first three waves; wave sums, then their totals in order
        __shared__ double wsum[3][2];
        n0 = wave_sum(n0);
        n1 = wave_sum(n1);
        if ((tid & 63) == 0 && tid < 192) {
            wsum[tid >> 6][0] = n0;
            wsum[tid >> 6][1] = n1;
        }
        __syncthreads();
        if (tid == 0) {
            const size_t pb = (size_t)col * a.nslots + blk;
            a.partial[2 * pb] = wsum[0][0] + wsum[1][0] + wsum[2][0];
            a.partial[2 * pb + 1] = wsum[0][1] + wsum[1][1] + wsum[2][1];
        }
    }
}

}  // namespace bri

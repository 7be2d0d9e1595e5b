// stencil_rows_kernel: the Brillouin stencil on four right-hand sides per block with the colour
// transport fed by lane-row broadcasts.
//
// A wave is four rows of 16 lanes.  A row holds one site, its 16 lanes the four spins of four right-hand
// sides, so that the whole row multiplies by one 3x3 link: lane e < 9 of the row holds link entry e, and
// every multiply-add takes it as a row_newbcast operand (in FP64 at full rate, in FP32 at half the plain
// rate, and without a register copy).  Lane = site, as in the kernels above, loads each link once per lane
// and pair of right-hand sides and each neighbour spinor once per displacement, and the vector-memory
// path holds it; here a link is one 16-lane operand for 16 spinor components.
//
// A block of twelve waves owns 48 sites, whole x-lines, and walks the 27 groups of equal (d_y, d_z, d_t).
// Per group it stages in LDS the group's neighbour lines of the four right-hand sides and the three
// slabs (d_x = -1, 0, +1) of 27 link entries, as coalesced line loads, and serves the three d_x from them.
// LDS holds [component][site] with an odd pitch: a row's 16 lanes (components 3 apart) and its nine link
// lanes then fall in distinct banks.  Two buffers alternate.  FP64 (118 KB: a block per CU, three waves
// a SIMD) keeps the staged registers few: a group's operands are read when they are used.  FP32 has
// the registers to read them a group ahead and to have the loads of two groups in flight.
//
// The weights of a group are a_m, c_m on d_x = 0 and a_m / 2, c_m / 4 on d_x = +-1 (the Laplacian and
// derivative weights halve and quarter with each hop).  With chi = W psi of the three neighbours,
//   s = chi(+) + chi(-),  delta = chi(+) - chi(-),  u = chi(0) + s/2,  v = chi(0) + s/4,
// the group adds a_m u + c_m (d_y gamma_2 + d_z gamma_3 + d_t gamma_4) v + (c_m / 4) gamma_1 delta.
// gamma_1 and gamma_2 exchange the spins 0-3, 1-2, gamma_3 and gamma_4 the spins 0-2, 1-3, so each lane
// keeps three sums of its own spin (unchanged, to be sent to spin 3 - s, to spin s ^ 2) and the spins
// are exchanged once, after the last group.
//
// What holds it is the latency of a group, from barrier to barrier.  24^3x48, 12 right-hand sides, line tiles ->
// here: FP64 11.0 -> 8.7 ms, FP32 6.8 -> 5.7 (reading when used: 6.6), bfloat16 links 6.2 -> 5.65; FP64 with the
// operands a group ahead spills and takes 35 ms.
#pragma once

#include "stencil_core.hpp"

namespace bri {

constexpr int ROWS_RHS = 4;              // right-hand sides per block
constexpr int ROWS_SITES = 48;           // sites per block
constexpr int ROWS_PITCH = 49;           // entries per component in LDS
constexpr int ROWS_PSI = 12 * ROWS_RHS;  // staged spinor components
constexpr int ROWS_LNK = 27;             // staged link entries: 3 slabs x 9
constexpr int ROWS_THREADS = 16 * ROWS_SITES;

// quad permutation of the lanes (spins) of a quad
template <int CTRL> __device__ __forceinline__ float quad_perm(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ double quad_perm(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// c += w p (ADJ: w^dag p) with entry e of the link in lane e of the row: 36 multiply-adds, the link
// operand broadcast within each row of 16 lanes.  The wait states before the first one cover a link
// register last written by a vector instruction (a DPP operand may be read two states after that).
// The six sums take turns, so that a wave's dependent multiply-adds are six issues apart.
#define BRI_RB(op, acc, sg, w, p, n) op " " acc ", " sg w ", " p " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n"
// the six sums += (entries n0, n1, n2 of the link) * one spinor component (pr, pi); ADJ: conjugated
#define BRI_RB_COL(op, pr, pi, sr, si, n0, n1, n2)                                                           \
    BRI_RB(op, "%0", "", "%6", pr, n0) BRI_RB(op, "%1", "", "%6", pi, n0) BRI_RB(op, "%2", "", "%6", pr, n1) \
        BRI_RB(op, "%3", "", "%6", pi, n1) BRI_RB(op, "%4", "", "%6", pr, n2) BRI_RB(op, "%5", "", "%6", pi, n2) \
            BRI_RB(op, "%0", sr, "%7", pi, n0) BRI_RB(op, "%1", si, "%7", pr, n0) BRI_RB(op, "%2", sr, "%7", pi, n1) \
                BRI_RB(op, "%3", si, "%7", pr, n1) BRI_RB(op, "%4", sr, "%7", pi, n2) BRI_RB(op, "%5", si, "%7", pr, n2)
#define BRI_RB_ASM(op)                                                                                               \
    if constexpr (ADJ)                                                                                               \
        asm("s_nop 1\n" BRI_RB_COL(op, "%8", "%9", "", "-", 0, 1, 2) BRI_RB_COL(op, "%10", "%11", "", "-", 3, 4, 5)  \
                BRI_RB_COL(op, "%12", "%13", "", "-", 6, 7, 8)                                                       \
            : "+v"(c[0].x), "+v"(c[0].y), "+v"(c[1].x), "+v"(c[1].y), "+v"(c[2].x), "+v"(c[2].y)                     \
            : "v"(w.x), "v"(w.y), "v"(p[0].x), "v"(p[0].y), "v"(p[1].x), "v"(p[1].y), "v"(p[2].x), "v"(p[2].y));     \
    else                                                                                                             \
        asm("s_nop 1\n" BRI_RB_COL(op, "%8", "%9", "-", "", 0, 3, 6) BRI_RB_COL(op, "%10", "%11", "-", "", 1, 4, 7)  \
                BRI_RB_COL(op, "%12", "%13", "-", "", 2, 5, 8)                                                       \
            : "+v"(c[0].x), "+v"(c[0].y), "+v"(c[1].x), "+v"(c[1].y), "+v"(c[2].x), "+v"(c[2].y)                     \
            : "v"(w.x), "v"(w.y), "v"(p[0].x), "v"(p[0].y), "v"(p[1].x), "v"(p[1].y), "v"(p[2].x), "v"(p[2].y))

template <bool ADJ> __device__ __forceinline__ void row_transport(double2 (&c)[3], const double2 &w, const double2 (&p)[3]) {
    BRI_RB_ASM("v_fmac_f64_dpp");
}
template <bool ADJ> __device__ __forceinline__ void row_transport(float2 (&c)[3], const float2 &w, const float2 (&p)[3]) {
    BRI_RB_ASM("v_fmac_f32_dpp");
}

// the stored form of a link entry as the compute type
__device__ __forceinline__ double2 link_value(const double2 &v) { return v; }
__device__ __forceinline__ float2 link_value(const float2 &v) { return v; }
__device__ __forceinline__ float2 link_value(uint32_t u) {
    return make_float2(__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u));
}

// FP64: three waves a SIMD leave 168 registers each
template <class LS, bool DAG, int MODE>
__global__ __launch_bounds__(ROWS_THREADS) __attribute__((amdgpu_waves_per_eu(sizeof(typename LS::R) == 8 ? 3 : 2)))
void stencil_rows_kernel(StencilArgs a) {
    using R = typename LS::R;
    using C = typename Cx<R>::T;
    using S = typename LS::store_t;
    constexpr bool AHEAD = sizeof(R) == 4;           // operands and loads a group further ahead
    constexpr int SETS = AHEAD ? 2 : 1;              // groups whose loads are in flight
    constexpr int PITCH = ROWS_PITCH;
    constexpr int NP = ROWS_PSI / 16, NL = 2;        // staged elements per thread: 16 components a pass
    extern __shared__ __align__(16) unsigned char rows_lds[];

    int blk, grp;
    tile_and_group(a.nslots, a.xcd_remap, blk, grp, a.reverse);
    const int col0 = grp * ROWS_RHS;
    const int nlive = a.ncol - col0 < ROWS_RHS ? a.ncol - col0 : ROWS_RHS;
    if (nlive <= 0) return;
    {
        bool any = false;
        for (int q = 0; q < nlive; ++q) any |= !col_done<MODE>(a, col0 + q);
        if (!any) return;
    }

    const int Lx = a.g.L[0], Ly = a.g.L[1], Lz = a.g.L[2], Lt = a.g.L[3];
    const size_t V = (size_t)a.g.V;
    int y0, z, t;
    {
        const int per_col = a.coly * a.colz * Lt;
        const int colm = blk / per_col;
        int rem = blk - colm * per_col;
        const int ncy = a.nb[1] / a.coly;
        const int yy = rem % a.coly;
        rem /= a.coly;
        y0 = ((colm % ncy) * a.coly + yy) * a.tile[1];
        z = (colm / ncy) * a.colz + rem % a.colz;
        t = rem / a.colz;
    }
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = lane >> 4, n = lane & 15;

    // staging: thread -> site sm of the tile and the components sc, sc + 16, ...
    const int sc = tid / ROWS_SITES, sm = tid - sc * ROWS_SITES;
    const int sline = sm / Lx, sx = sm - sline * Lx, sy = y0 + sline;
    const unsigned plane = (unsigned)Lx * Ly, vol3 = plane * Lz;
    const C *__restrict__ in = (const C *)a.in + (size_t)col0 * 12 * V;
    const S *__restrict__ W = (const S *)a.W;
    const unsigned own_site = (unsigned)sx + (unsigned)sy * Lx + (unsigned)z * plane + (unsigned)t * vol3;

    // two buffers of [75][PITCH] entries
    constexpr int BUF = (ROWS_PSI + ROWS_LNK) * PITCH;
    C *const lds = (C *)rows_lds;

    // every thread loads in every pass, the surplus ones an element of the last component again
    R rpx[SETS][NP], rpy[SETS][NP];
    S rl[SETS][NL];
    unsigned po[NP], lo[NL];
#pragma unroll
    for (int k = 0; k < NP; ++k) po[k] = (unsigned)min(sc + k * 16, 12 * nlive - 1) * (unsigned)V;
#pragma unroll
    for (int k = 0; k < NL; ++k) lo[k] = (unsigned)min(sc + k * 16, ROWS_LNK - 1) * (unsigned)V;
    auto load = [&](auto set, int g) {
        constexpr int A = decltype(set)::value;
        const int dy = g % 3 - 1, dz = (g / 3) % 3 - 1, dt = g / 9 - 1;
        int yy = sy + dy;
        yy = yy < 0 ? yy + Ly : (yy >= Ly ? yy - Ly : yy);
        int zz = z + dz, tt = t + dt;
        zz = zz < 0 ? zz + Lz : (zz >= Lz ? zz - Lz : zz);
        tt = tt < 0 ? tt + Lt : (tt >= Lt ? tt - Lt : tt);
        const unsigned site = (unsigned)sx + (unsigned)yy * Lx + (unsigned)zz * plane + (unsigned)tt * vol3;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const C v = in[po[k] + site];
            rpx[A][k] = v.x;
            rpy[A][k] = v.y;
        }
        // own terms (g <= 13): slabs 3g.. at the own site; partner terms: slabs 78 - 3g.. at the
        // neighbour's line.  Group 13 holds d = (-1,0,0,0) and its opposite, slab 39: the last three
        // slabs are staged (37, 38, 39), slab 39 last.
        const S *wl = W + (size_t)(g < 13 ? 27 * g : g == 13 ? 333 : 27 * (26 - g)) * V;
        const unsigned ls = g <= 13 ? own_site : site;
#pragma unroll
        for (int k = 0; k < NL; ++k) rl[A][k] = wl[lo[k] + ls];
    };
    unsigned wpo[NP], wlo[NL];  // where they go in a buffer (surplus threads write an element a second time)
#pragma unroll
    for (int k = 0; k < NP; ++k) wpo[k] = __umul24(min(sc + k * 16, 12 * nlive - 1), PITCH) + sm;
#pragma unroll
    for (int k = 0; k < NL; ++k) wlo[k] = __umul24(ROWS_PSI + min(sc + k * 16, ROWS_LNK - 1), PITCH) + sm;
    auto stage = [&](auto set, C *to) {
        constexpr int A = decltype(set)::value;
#pragma unroll
        for (int k = 0; k < NP; ++k) to[wpo[k]] = cmake<C>(rpx[A][k], rpy[A][k]);
#pragma unroll
        for (int k = 0; k < NL; ++k) to[wlo[k]] = link_value(rl[A][k]);
    };

    // compute: the site of this row, its x-neighbours in the tile's line
    const int m0 = wv * 4 + row;
    int mm, mp;
    {
        const int x = m0 % Lx;
        mm = x == 0 ? m0 + Lx - 1 : m0 - 1;
        mp = x == Lx - 1 ? m0 - x : m0 + 1;
    }
    const int pbase = n * 3 * PITCH, wbase = (ROWS_PSI + (n < 9 ? n : 8)) * PITCH;
    const R g1 = (n & 2) ? (R)-1 : (R)1;                         // gamma_1: i g1
    const R g2 = ((n & 3) == 1 || (n & 3) == 2) ? (R)1 : (R)-1;  // gamma_2
    const R g3 = ((n & 3) == 0 || (n & 3) == 3) ? (R)1 : (R)-1;  // gamma_3: i g3

    C A0[3], F3[3], F2[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) A0[c] = F3[c] = F2[c] = cmake<C>((R)0, (R)0);

    // The operands of a group from its buffer.  Kinds of groups: 0 own links (at the site), 1 partner
    // links (at the neighbour, daggered), 2 group 13 (own for d_x = -1, partner for +1, both of the last
    // slab).
    C pm[3], pc[3], pp[3], wm, wc, wp;
    auto read_m = [&](auto kind, const C *buf) {
        constexpr int K = decltype(kind)::value;
        wm = K == 1 ? buf[wbase + 18 * PITCH + mm] : buf[wbase + (K == 2 ? 18 * PITCH : 0) + m0];
#pragma unroll
        for (int c = 0; c < 3; ++c) pm[c] = buf[pbase + c * PITCH + mm];
    };
    auto read_p = [&](auto kind, const C *buf) {
        constexpr int K = decltype(kind)::value;
        wp = K == 0 ? buf[wbase + 18 * PITCH + m0] : buf[wbase + (K == 2 ? 18 * PITCH : 0) + mp];
#pragma unroll
        for (int c = 0; c < 3; ++c) pp[c] = buf[pbase + c * PITCH + mp];
    };
    auto read_c = [&](auto kind, const C *buf) {
        if constexpr (decltype(kind)::value != 2) wc = buf[wbase + 9 * PITCH + m0];
#pragma unroll
        for (int c = 0; c < 3; ++c) pc[c] = buf[pbase + c * PITCH + m0];
    };
    // Group g of this kind, the next one of kind knext; flat: d_z = d_t = 0.  A weight that is zero adds nothing, or
    // an infinite neighbour would reach spins that its displacement does not couple (0 * inf): flat groups have
    // no F2 terms, and those of d_y = 0 skip the one of F3 (a branch a term: FP64 8% slower, FP32 4%).  The
    // barriers around the scheduler keep the LDS reads and the staging where they are written: hoisted, their
    // registers spill.
    auto step = [&](auto kind, auto knext, auto set, auto flat, int g) {
        constexpr int K = decltype(kind)::value, FLAT = decltype(flat)::value;
        C *const cur = lds + (g & 1) * BUF, *const next = lds + ((g + 1) & 1) * BUF;
        if constexpr (!AHEAD) {
            __syncthreads();  // group g is staged, and every wave is done with the other buffer
            read_m(kind, cur);
            read_p(kind, cur);
            if (g < 26) stage(set, next);
            if (g < 25) load(set, g + 2);
        }
        const int dy = g % 3 - 1, dz = (g / 3) % 3 - 1, dt = g / 9 - 1;
        // a_h = -2^-(h+3), c_h = (16/27) 4^-h
        const int h = (dy != 0) + (dz != 0) + (dt != 0);
        const R am = scale_pow2((R)-0.125, -h);
        const R cm = scale_pow2((R)((DAG ? -16.0 : 16.0) / 27.0), -2 * h);
        const R cx = (R)0.25 * cm * g1;
        C s[3], u[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] = cmake<C>((R)0, (R)0);
        if constexpr (!AHEAD) __builtin_amdgcn_sched_barrier(0);
        row_transport<K == 1>(s, wm, pm);  // chi(-)
        if constexpr (!AHEAD) {
            __builtin_amdgcn_sched_barrier(0);
            read_c(kind, cur);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) axpy_ic(F3[c], (R)-2 * cx, s[c]);  // gamma_1 (chi(+) - chi(-)): -2 chi(-) here, + s below
        if constexpr (!AHEAD) __builtin_amdgcn_sched_barrier(0);
        row_transport<K != 0>(s, wp, pp);  // s
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (AHEAD) {
            // every wave holds all operands of group g, and group g + 1 is staged: its reads run under the
            // rest of this group
            __syncthreads();
            if (g < 25) stage(set, cur);  // group g + 2
            read_m(knext, next);
            read_p(knext, next);
            if (g < 23) load(set, g + 4);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            axpy_ic(F3[c], cx, s[c]);
            u[c] = cmake<C>((R)0.5 * s[c].x, (R)0.5 * s[c].y);
        }
        if constexpr (K != 2) {
            const R cy = cm * (R)dy * g2, cz = cm * (R)dz * g3, ct = cm * (R)dt;
            C vy[3];
            row_transport<K == 1>(u, wc, pc);
            if constexpr (AHEAD) {
                __builtin_amdgcn_sched_barrier(0);
                read_c(knext, next);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const C v = cmake<C>(fma((R)-0.25, s[c].x, u[c].x), fma((R)-0.25, s[c].y, u[c].y));
                axpy_c(A0[c], am, u[c]);
                if constexpr (FLAT == 0) {
                    axpy_c(F2[c], ct, v);
                    axpy_ic(F2[c], cz, v);
                }
                vy[c] = v;
            }
            if (dy) {
#pragma unroll
                for (int c = 0; c < 3; ++c) axpy_c(F3[c], cy, vy[c]);
            }
        } else {
            const R diag = (R)a.diag;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                axpy_c(A0[c], am, u[c]);
                axpy_c(A0[c], diag, pc[c]);
            }
            if constexpr (AHEAD) {
                __builtin_amdgcn_sched_barrier(0);
                read_c(knext, next);
            }
        }
    };

    using Own = std::integral_constant<int, 0>;
    using Partner = std::integral_constant<int, 1>;
    using Centre = std::integral_constant<int, 2>;
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, SETS - 1>;
    using Deep = std::integral_constant<int, 0>;
    using Flat = std::integral_constant<int, 1>;
    load(Even{}, 0);
    if constexpr (AHEAD) {
        load(Odd{}, 1);
        stage(Even{}, lds);
        load(Even{}, 2);
        stage(Odd{}, lds + BUF);
        load(Odd{}, 3);
        __syncthreads();  // groups 0 and 1 are staged
        read_m(Own{}, lds);
        read_p(Own{}, lds);
        read_c(Own{}, lds);
#pragma unroll 1
        for (int g = 0; g < 12; g += 2) {
            step(Own{}, Own{}, Even{}, Deep{}, g);
            step(Own{}, Own{}, Odd{}, Deep{}, g + 1);
        }
        step(Own{}, Centre{}, Even{}, Flat{}, 12);
        step(Centre{}, Partner{}, Odd{}, Flat{}, 13);
        step(Partner{}, Partner{}, Even{}, Flat{}, 14);
#pragma unroll 1
        for (int g = 15; g < 27; g += 2) {  // (the reads of a next group after the last are unused)
            step(Partner{}, Partner{}, Odd{}, Deep{}, g);
            step(Partner{}, Partner{}, Even{}, Deep{}, g + 1);
        }
    } else {
        stage(Even{}, lds);
        load(Even{}, 1);
#pragma unroll 1
        for (int g = 0; g < 12; ++g) step(Own{}, Own{}, Even{}, Deep{}, g);
        step(Own{}, Centre{}, Even{}, Flat{}, 12);
        step(Centre{}, Partner{}, Even{}, Flat{}, 13);
        step(Partner{}, Partner{}, Even{}, Flat{}, 14);
#pragma unroll 1
        for (int g = 15; g < 27; ++g) step(Partner{}, Partner{}, Even{}, Deep{}, g);
    }

    // the spin exchange, then the results through LDS into the staging's (component, site) order, in the
    // buffer that no wave still reads (read ahead, group 26 was read before the last barrier; the reads
    // of a group 27 are of the other buffer)
    C *const res = AHEAD ? lds : lds + BUF;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        C v = A0[c];
        v.x += quad_perm<0x1b>(F3[c].x) + quad_perm<0x4e>(F2[c].x);
        v.y += quad_perm<0x1b>(F3[c].y) + quad_perm<0x4e>(F2[c].y);
        res[(n * 3 + c) * PITCH + m0] = v;
    }
    __syncthreads();
    double n0[ROWS_RHS], n1[ROWS_RHS];
#pragma unroll
    for (int q = 0; q < ROWS_RHS; ++q) {
        n0[q] = n1[q] = 0.0;
        if (q >= nlive || col_done<MODE>(a, col0 + q) || sc >= 12) continue;
        C v = res[(q * 12 + sc) * PITCH + sm];
        if (a.g.csw != 0.0)
            clover_row<LS>(v, W + (size_t)LINK_SLAB_ENTRIES * V, in + (size_t)q * 12 * V, sc, own_site, (unsigned)V);
        epilogue<MODE, C, R>(a, col0 + q, sc, own_site, (unsigned)V, v, n0[q], n1[q], col_alpha<MODE>(a, col0 + q));
    }
    if constexpr (MODE == EPI_NORMS || MODE == EPI_CG_R) {
        // deterministic: wave sums, then the wave totals in order
        __shared__ double wsum[ROWS_THREADS / 64][ROWS_RHS][2];
#pragma unroll
        for (int q = 0; q < ROWS_RHS; ++q) {
            const double s0 = wave_sum(n0[q]), s1 = MODE == EPI_NORMS ? wave_sum(n1[q]) : 0.0;
            if (lane == 0) {
                wsum[wv][q][0] = s0;
                wsum[wv][q][1] = s1;
            }
        }
        __syncthreads();
        if (tid < nlive && !col_done<MODE>(a, col0 + tid)) {
            double s0 = 0.0, s1 = 0.0;
            for (int w = 0; w < ROWS_THREADS / 64; ++w) {
                s0 += wsum[w][tid][0];
                s1 += wsum[w][tid][1];
            }
            const size_t pb = (size_t)(col0 + tid) * a.nslots + blk;
            a.partial[2 * pb] = s0;
            a.partial[2 * pb + 1] = s1;
        }
    }
}

}  // namespace bri

// Stencil launches: tile planning, default configurations, the dispatch to the per-variant
// instantiations (stencil_<precision>_<kernel>.hip) and the bri_apply / wil_apply entry points.
#include <algorithm>

#include "stencil.hpp"

namespace bri {

// one translation unit per (link precision, kernel) pair
hipError_t launch_f64_bri(const StencilArgs &, bool, int, const StencilConfig &, hipStream_t);
hipError_t launch_f64_wil(const StencilArgs &, bool, int, const StencilConfig &, hipStream_t);
hipError_t launch_f32_bri(const StencilArgs &, bool, int, const StencilConfig &, hipStream_t);
hipError_t launch_f32_wil(const StencilArgs &, bool, int, const StencilConfig &, hipStream_t);
hipError_t launch_bf16_bri(const StencilArgs &, bool, int, const StencilConfig &, hipStream_t);
hipError_t launch_bf16_wil(const StencilArgs &, bool, int, const StencilConfig &, hipStream_t);
hipError_t launch_f64_rows(const StencilArgs &, bool, int, hipStream_t);
hipError_t launch_f32_rows(const StencilArgs &, bool, int, hipStream_t);
hipError_t launch_bf16_rows(const StencilArgs &, bool, int, hipStream_t);

// A 64-site tile that divides the lattice.  Column traversal: tile
// tile[0] x tile[1] x 1 x 1 with colz | Lz.  Otherwise x first (coalescing),
// then y, z, t.
static int plan_tile_base(const Geom &g, const StencilConfig &cfg, int tile[4], int nb[4]) {
    if (g.V % 64) return BRI_EINVAL;
    if (cfg.colz <= 0 && cfg.coly > 1) return BRI_EINVAL;  // y-blocked columns need the column traversal
    if (cfg.variant == VAR_TSTREAM) {
        // t-streaming: an xyz tile of STREAM_THREADS sites and chunks of tile[3] t-slices
        if (cfg.rpt != 0) return BRI_EINVAL;
        int prod = 1;
        for (int mu = 0; mu < 4; ++mu) {
            if (cfg.tile[mu] < 1 || g.L[mu] % cfg.tile[mu]) return BRI_EINVAL;
            if (mu < 3) prod *= cfg.tile[mu];
        }
        if (prod != STREAM_THREADS) return BRI_EINVAL;
        for (int mu = 0; mu < 4; ++mu) {
            tile[mu] = cfg.tile[mu];
            nb[mu] = g.L[mu] / tile[mu];
        }
        return BRI_OK;
    }
    if (cfg.colz > 0) {
        const int tx = cfg.tile[0], ty = cfg.tile[1];
        if (tx < 1 || ty < 1 || tx * ty != 64 || g.L[0] % tx || g.L[1] % ty || g.L[2] % cfg.colz) return BRI_EINVAL;
        tile[0] = tx;
        tile[1] = ty;
        tile[2] = tile[3] = 1;
        nb[0] = g.L[0] / tx;
        nb[1] = g.L[1] / ty;
        nb[2] = g.L[2];
        nb[3] = g.L[3];
        if (cfg.coly < 0 || (cfg.coly > 0 && nb[1] % cfg.coly)) return BRI_EINVAL;
        return BRI_OK;
    }
    if (cfg.tile[0] > 0) {
        int prod = 1;
        for (int mu = 0; mu < 4; ++mu) {
            if (cfg.tile[mu] < 1 || g.L[mu] % cfg.tile[mu]) return BRI_EINVAL;
            prod *= cfg.tile[mu];
        }
        if (prod != 64) return BRI_EINVAL;
        for (int mu = 0; mu < 4; ++mu) {
            tile[mu] = cfg.tile[mu];
            nb[mu] = g.L[mu] / tile[mu];
        }
        return BRI_OK;
    }
    int rem = 64;
    for (int mu = 0; mu < 4; ++mu) {
        int t = 1;
        while (rem % (2 * t) == 0 && g.L[mu] % (2 * t) == 0 && 2 * t <= rem && 2 * t <= 16) t *= 2;
        tile[mu] = t;
        rem /= t;
    }
    for (int mu = 0; mu < 4 && rem > 1; ++mu)
        while (rem > 1 && g.L[mu] % (tile[mu] * 2) == 0) {
            tile[mu] *= 2;
            rem /= 2;
        }
    if (rem != 1) return BRI_EINVAL;
    for (int mu = 0; mu < 4; ++mu) nb[mu] = g.L[mu] / tile[mu];
    return BRI_OK;
}

// the tile plan, and for the x-line kernel the requirement that a tile spans whole x-lines
int plan_tile(const Geom &g, const StencilConfig &cfg, int tile[4], int nb[4]) {
    const int rc = plan_tile_base(g, cfg, tile, nb);
    if (rc != BRI_OK) return rc;
    if (cfg.variant == VAR_XLINE && (tile[0] != g.L[0] || cfg.rpt == 1 || cfg.rpt > 4)) return BRI_EINVAL;
    if (cfg.variant == VAR_MFMA && (cfg.rpt < 1 || cfg.rpt > 4)) return BRI_EINVAL;
    if (cfg.variant < VAR_STANDARD || cfg.variant > VAR_MFMA) return BRI_EINVAL;
    return BRI_OK;
}

// tiles of `n` whole x-lines, the last tile of a (z, t) plane possibly with fewer
static int line_tiles(const Geom &g, int n) { return (g.L[1] + n - 1) / n * g.L[2] * g.L[3]; }

int stencil_slots(const Geom &g, const StencilConfig &cfg) {
    return cfg.small > 0 ? g.V / 16
           : cfg.rows > 0 || cfg.lines > 0 ? line_tiles(g, cfg.rows > 0 ? cfg.rows : cfg.lines)
                                           : g.V / 64;
}

// The solvers apply D and D^dag in turn.  Links larger than the 256 MiB last-level cache, but not by much,
// are read by each in the order in which the other has pushed them out; with the adjoint walking tiles and
// slabs backwards each finds what the other read last.  16 iterations of the multi-shift CG: 16^4 (360
// MiB) 3.35 -> 3.23 ms, 12^3x32 (303) 3.34 -> 3.23; 24^2x12x16 (607) 5.89 -> 5.95, 32^3x64 5% slower, and
// below the cache's size (12^3x24, 227) no difference.
static bool reverse_pays(const Geom &g, int prec) {
    const long long bytes = 360LL * g.V * (prec == BRI_F64 ? 16 : prec == BRI_F32 ? 8 : 4);
    return bytes > 256LL << 20 && bytes <= 512LL << 20;
}

int stencil_launch(StencilArgs a, int prec, bool dag, int mode, const StencilConfig &cfg, hipStream_t st) {
    if (a.ncol < 1 || a.ncol > 65535) return BRI_EINVAL;
    int rc = BRI_OK;
    if (cfg.rows > 0 || cfg.lines > 0) {
        const int n = cfg.rows > 0 ? cfg.rows : cfg.lines;
        a.tile[0] = a.g.L[0];
        a.tile[1] = n;
        a.tile[2] = a.tile[3] = 1;
        a.nb[0] = 1;
        a.nb[1] = (a.g.L[1] + n - 1) / n;
        a.nb[2] = a.g.L[2];
        a.nb[3] = a.g.L[3];
    } else if (cfg.small == 0) {
        rc = plan_tile(a.g, cfg, a.tile, a.nb);
    }
    if (rc != BRI_OK) return rc;
    a.colz = cfg.colz;
    a.coly = cfg.coly > 0 ? cfg.coly : 1;
    a.xcd_remap = cfg.xcd_remap;
    a.nslots = stencil_slots(a.g, cfg);
    a.reverse = a.kind == KERN_BRI && dag && reverse_pays(a.g, prec);
    if (a.kind != KERN_BRI && a.kind != KERN_WIL) return BRI_EINVAL;
    const bool wil = a.kind == KERN_WIL;
    hipError_t e;
    if (cfg.rows > 0)
        e = wil                     ? hipErrorInvalidValue
            : prec == BRI_F64       ? launch_f64_rows(a, dag, mode, st)
            : prec == BRI_F32       ? launch_f32_rows(a, dag, mode, st)
            : prec == BRI_F32_BF16W ? launch_bf16_rows(a, dag, mode, st)
                                    : hipErrorInvalidValue;
    else if (prec == BRI_F64)
        e = wil ? launch_f64_wil(a, dag, mode, cfg, st) : launch_f64_bri(a, dag, mode, cfg, st);
    else if (prec == BRI_F32)
        e = wil ? launch_f32_wil(a, dag, mode, cfg, st) : launch_f32_bri(a, dag, mode, cfg, st);
    else if (prec == BRI_F32_BF16W)
        e = wil ? launch_bf16_wil(a, dag, mode, cfg, st) : launch_bf16_bri(a, dag, mode, cfg, st);
    else
        return BRI_EINVAL;
    return e == hipSuccess ? BRI_OK : (e == hipErrorInvalidValue ? BRI_EINVAL : BRI_EHIP);
}

// Column traversal when the lattice allows a 16 x 4 tile (two full 128-byte lines per row in
// FP64) and a column depth of 8 (or 4, 2) z-planes; lexicographic tiles otherwise, which
// measured faster than 8 x 8 or 4 x 16 columns (24^3 x 48: 1.86 against 2.04 ms).
static void default_traversal(const Geom &g, StencilConfig &c) {
    for (int mu = 0; mu < 4; ++mu) c.tile[mu] = 0;
    c.colz = 0;
    if (g.L[0] % 16 || g.L[1] % 4) return;
    for (int cz : {8, 4, 2}) {
        if (g.L[2] % cz) continue;
        c.tile[0] = 16;
        c.tile[1] = 4;
        c.colz = cz;
        return;
    }
}

// a large lattice whose x-lines fill whole rows of a 64-lane wave (the x-line kernels' default)
static bool xline_fits(const Geom &g) {
    return g.V / 64 >= 8192 && (g.L[0] == 16 || g.L[0] == 32 || g.L[0] == 64) && g.L[1] % (64 / g.L[0]) == 0;
}

// The default in terms of bri_stencil_cfg (64-site tiles); the tuned table holds Brillouin launches
// only, the Wilson stencil keeps the defaults.
StencilConfig tile_config(const Geom &g, int prec, int ncol, int kind) {
    StencilConfig c;
    default_traversal(g, c);
    c.xcd_remap = 1;
    if (ncol >= 2) {
        // link loads amortised over R right-hand sides per thread (a last, partial group of
        // columns is allowed); four waves still split each tile's displacements.  Below 4096
        // tiles (up to 16^4) more column groups keep the chip busy: R = 2 (FP64, and FP32 up to 8
        // columns) or 3 measured 5-40% faster than R = 4 at 8^4 and 16^4; at 24^3x48 R = 4 is
        // fastest (by up to 25% in FP32).
        c.nsplit = MRHS_SPLIT;
        if (ncol < 4)
            c.rpt = ncol;
        else if (g.V / 64 < 4096)
            c.rpt = (prec == BRI_F64 || ncol <= 8) ? 2 : 3;
        else
            c.rpt = (ncol % 4 == 0 || ncol % 3 != 0) ? 4 : 3;
        // large lattices whose x-lines fit a wave: whole-line tiles (Lx x 64/Lx) in columns of 4
        // z-slices (FP64: one tile row wide; FP32 and bfloat16 links: two), the column groups of
        // a tile run together (tile_and_group).  12 RHS at 32^3x64 measured 28.8-29.2 ms (FP64, R
        // = 2; 30.2 / 31.4 ms in columns of 8 / 16 z-slices; two rows wide the same time with 8%
        // more bytes fetched), 16.4 ms (FP32, R = 3; 16.8 ms one row wide, 17.4 ms with R = 4) and
        // 14.9 ms (bfloat16 links: the x-line kernel, one RHS per thread; 15.1 ms for the
        // multi-RHS kernel with R = 3).  Before the tiles' column groups ran together (each group
        // a separate pass over the lattice, re-reading every link) the same launches took 37.6 /
        // 18.5 / 18.7 ms.
        if (kind == KERN_BRI && ncol >= 3 && xline_fits(g)) {
            c.tile[0] = g.L[0];
            c.tile[1] = 64 / g.L[0];
            c.tile[2] = c.tile[3] = 1;
            c.xcd_remap = 1;
            c.colz = g.L[2] % 4 == 0 ? 4 : (g.L[2] % 2 == 0 ? 2 : 1);
            c.coly = prec != BRI_F64 && (g.L[1] / c.tile[1]) % 2 == 0 ? 2 : 1;
            if (prec == BRI_F32_BF16W) {
                c.variant = VAR_XLINE;
                c.rpt = 0;
            } else {
                c.rpt = prec == BRI_F64 ? 2 : 3;
            }
        }
    } else {
        // four waves split each tile's directions: fills the 1024 SIMDs on small lattices, and on
        // large ones keeps fewer tiles (and their link lines) in flight per XCD than two waves do
        c.rpt = 0;
        c.nsplit = 4;
        // large lattices whose x-lines fit a wave: the x-line kernel (one spinor load per three
        // x-displacements) on whole-line tiles in XCD-ordered columns of 4 z-slices and 8 (FP64)
        // or 16 tile rows, whose tiles run together with their y, z and t neighbours, where the
        // partner sites re-read the links.  At 32^3x64 it measured 3.59-3.63 / 2.00 / 1.47 ms
        // (FP64 / FP32 / bfloat16 links) against 4.17 / 2.21 / 1.71 ms for lexicographic tiles
        // (the fastest traversal without y-blocked columns) and 5.52 / 3.37 / 2.64 ms for the 16 x
        // 4 column traversal above; at 16^4 the kernels tie.
        if (kind == KERN_BRI && xline_fits(g)) {
            c.variant = VAR_XLINE;
            c.tile[0] = g.L[0];
            c.tile[1] = 64 / g.L[0];
            c.tile[2] = c.tile[3] = 1;
            const int rows = g.L[1] / c.tile[1];
            c.colz = g.L[2] % 4 == 0 ? 4 : (g.L[2] % 2 == 0 ? 2 : 1);
            const int widest = prec == BRI_F64 ? 8 : 16;
            c.coly = 1;
            for (int cy = widest; cy > 1; cy /= 2)
                if (rows % cy == 0) {
                    c.coly = cy;
                    break;
                }
            c.xcd_remap = 1;
        }
    }
    return c;
}

constexpr int SMALL_MAX_SITES = 16 * 1536;  // the small-lattice kernel's blocks of 16 sites

// Whole x-lines of at most 64 sites per wave.  Lines of 16, 32 or 64 sites fill the wave; other lengths
// leave lanes idle (24-site lines: 48 of 64), and still win over 64-site tiles that cut the lines: the
// x-neighbours come by lane moves, every load is one or a few full runs of sites, and the tile rows
// form columns.  One right-hand side, before -> now: 24^3x48 FP64 1967 -> 1275 us, FP32 1298 -> 700;
// 20x12x28x24 FP64 637 -> 300; 31x12x16x14 (extents whose only even tiles are 1 x 4 x 16 x 1) 879 -> 175;
// 36x16x29x26 (36 of 64 lanes) 1675 -> 1200.  Below half the lanes the cut tiles stay.
static bool lines_fit(const Geom &g, int *lines) {
    if (g.L[0] > 64) return false;
    int n = 64 / g.L[0];
    if (n > g.L[1]) n = g.L[1];
    if ((long long)line_tiles(g, n) * 32 > g.V) return false;
    *lines = n;
    return true;
}

// Columns of coly tile rows by colz z-planes: of the divisors, the cross-section with the smallest
// halo (lines around it that are read with it) among those of at most `cap` tiles.
static void line_columns(const Geom &g, int lines, int cap, StencilConfig &c) {
    const int rows = (g.L[1] + lines - 1) / lines;
    double best = 1e300;
    for (int cz = 1; cz <= g.L[2] && cz <= cap; ++cz)
        for (int cy = 1; cy <= rows && cy * cz <= cap; ++cy) {
            if (g.L[2] % cz || rows % cy) continue;
            const double halo = (cz + 2.0) * (cy * lines + 2.0) / ((double)cz * cy * lines);
            if (halo < best) {
                best = halo;
                c.colz = cz;
                c.coly = cy;
            }
        }
}

constexpr int CUS = 256;

// The four-right-hand-side kernel: blocks of exactly 48 sites in whole x-lines, one block a CU, 50 us (FP32 and
// bfloat16 links 35) however full the chip is: a last round of few blocks and groups with empty places cost as
// much as full ones.  The sites and right-hand sides have to fill more than three quarters of its rounds in
// FP64, five sixths in FP32.  Above the line, the better of line and cut tiles -> this kernel: FP64 24x20x12x6
// x 4 (94% full) 187 -> 164 us, 12x4x6x20 x 7 (82%) 58 -> 54, 12x8x8x8 x 8 (100%) 66 -> 54; FP32 24x4x12x16 x 8
// (100%) 126 -> 106, 12^3x24 x 4 (84%) 149 -> 139, bfloat16 links 48x16x4x12 x 4 (100%) 118 -> 105.  Below it:
// FP64 24x4x8x8 x 4 (50%) 40 -> 51, 48x2x12x24 x 4 (75%) 142 -> 161, 24x8x12x18 x 3 (63%) 190 -> 202; FP32
// 12x8x12x12 x 4 (56%) 61 -> 70, bfloat16 links 12x20x16x8 x 4 (83%) 84 -> 104.
// Groups of four that are full, or in FP64 lack one (24^3x48 x 7: FP64 6.7 -> 5.6 ms, FP32 4.0 -> 3.7, bfloat16
// links slower); beyond four rounds, where the other tiles slow down too, the empty place does not count
// (24x24x18x28 x 3 1460 -> 1310 us), nor in FP64's single round of more than 170 blocks (192: 24x8x4x12 x 3
// 59 -> 51 us, 48x4x8x6 x 4 72 -> 52; 160: 24x4x10x4 x 8 45 -> 51).  Blocks with idle rows lose (20-site lines:
// FP32 650 against 1120 us), and so do lines of 16 and 32 sites, which the x-line and standard kernels fill
// (16^3x64 x 12: FP64 3.6 against 3.7 ms).  The kernel's 32-bit offsets reach over the 48 staged components.
static bool rows_fit(const Geom &g, int prec, int ncol) {
    const int Lx = g.L[0];
    if (Lx != 12 && Lx != 24 && Lx != 48) return false;
    if (g.L[1] % (48 / Lx) || g.V > 0xffffffffLL / 48) return false;
    if (ncol % 4 && !(prec == BRI_F64 && ncol % 4 == 3)) return false;
    if (prec != BRI_F64 && g.V / 48 < CUS) return false;
    const long long tiles = g.V / 48, groups = (ncol + 3) / 4, rounds = (tiles * groups + CUS - 1) / CUS;
    if (rounds == 1 && prec == BRI_F64) return 3 * tiles * groups > 2 * CUS;
    const long long work = tiles * (rounds > 4 ? 4 * groups : ncol);
    return prec == BRI_F64 ? work > 3 * CUS * rounds : 3 * work > 10 * CUS * rounds;
}

bool forms_alpha(const StencilConfig &cfg, int ndots) {
    if (cfg.variant == VAR_TSTREAM || cfg.variant == VAR_MFMA || cfg.rows > 0) return false;
    return ndots <= MAX_DOTS && (cfg.small > 0 || cfg.rpt == 0);
}

// The blocks of a launch on `tiles` tiles, and how many of them the chip holds at once: two a CU in FP64
// (registers), one with the sums of several right-hand sides per thread in LDS; in FP32 four (x-line) or five,
// three, two and one with two, three and four per thread.
static long long launch_blocks(long long tiles, int ncol, const StencilConfig &c) {
    const int r = c.rpt > 1 ? c.rpt : 1;
    return tiles * ((ncol + r - 1) / r);
}
static int resident_blocks(int prec, const StencilConfig &c) {
    const int f32[5] = {c.variant == VAR_XLINE ? 4 : 5, 5, 3, 2, 1};
    return CUS * (prec != BRI_F64 ? f32[c.rpt] : c.rpt > 1 ? 1 : 2);
}

// The launch on tiles of n whole x-lines that leave lanes idle against the one on the cut tiles (c), which have a
// site on every lane: whether the cut tiles stay.  What decides is whether they hold whole x-lines too (4-, 8-
// and 16-site lines stacked over y, z and t), and in how long runs of consecutive sites; below, cut -> line
// tiles, one right-hand side where no number is given.
static bool cut_stays(const Geom &g, int prec, int ncol, int kind, const StencilConfig &c, const StencilConfig &line) {
    // (as plan_tile and the 16 x 4 columns choose them: powers of two up to 16, x first)
    int run = 1;
    bool whole = true;
    for (int mu = 0, all = 1; mu < 4 && all; ++mu) {
        const int pow2 = g.L[mu] & -g.L[mu], t = std::min({pow2, 16, 64 / run});
        all = t == g.L[mu];
        if (mu == 0) whole = all;
        run *= t;
    }
    const long long cut = g.V / 64, tiles = line_tiles(g, line.lines);
    const bool three_quarters = 4LL * g.V >= 3LL * 64 * tiles, most = 8LL * g.V >= 7LL * 64 * tiles,
               nine_tenths = 10LL * g.V >= 9LL * 64 * tiles;
    if (kind == KERN_WIL) {
        // Batches on whole lines, or on runs of four sites or more unless the lines use nine lanes in ten as well
        // (24^3x48 x 12: FP64 2.79 -> 3.27 ms; 12^3x24 x 3: FP32 21 -> 28 us; 20x12x28x24, 95%, 1.2 to 1.4
        // times faster on lines); shorter runs gain 1.1 to 13 times (6x16x12x48 x 9 with bfloat16 links loses,
        // 68 -> 80 us).  Two-site lines are whole either way: the cut tiles stay where they divide over the 8 XCDs
        // (2x20x32x64 FP64 x 3 67 -> 95 us, 2x16x40x8 FP32 x 9 16 -> 30; else 2x50x48x12 bfloat16 links x 6 117 ->
        // 53), and where they hold four lines or more in y and one lane in eight idles (2x40x28x14 x 8 30 -> 47).
        if (ncol > 1 && g.L[0] == 2) return cut % 8 == 0 || (!most && g.L[1] % 4 == 0);
        if (ncol > 1) return g.L[0] % 4 == 0 && (whole || !nine_tenths);
        // One right-hand side, bound by HBM or latency: whole x-lines either way (2x40x14x28 FP32 6.4 -> 8.9 us,
        // 8x20x20x32 bfloat16 links 8% slower), runs of 16 (48-site lines, 48x6x8x28 FP32 10.2 -> 12.8 us), and
        // where a second block a CU starts (24x6x16x6 FP64 5.6 -> 6.6 us).  Shorter runs gain, 24^3x48 FP64
        // 177 -> 168 us.
        return (!most && (whole || run >= 16)) || (cut <= CUS && tiles > CUS);
    }
    // The cut tiles in one round of resident blocks and the line tiles in more: FP64 24x24x6x4 x 2 48 -> 60 us,
    // 8x8x8x32 x 3 56 -> 63, bfloat16 links with idle lanes 48x2x24x6 x 4 49 -> 59.  (FP32 gains all the same,
    // 64x20x2x16 x 2 1.3 times, and so do shorter runs.)
    if (run >= 8 && (prec == BRI_F64 || (prec == BRI_F32_BF16W && ncol > 1 && !most)) &&
        launch_blocks(cut, ncol, c) <= resident_blocks(prec, c) &&
        launch_blocks(tiles, ncol, line) > resident_blocks(prec, line))
        return true;
    // Both whole lines, seven lanes in eight work (nine in ten for a batch of nine or more, 16x14x8x32 FP32 x 12
    // 435 -> 497 us; 8x28x40x16 x 5 615 -> 539): only one right-hand side in FP64 up to 512 tiles, where the order
    // of the tiles alone differs (16x24x18x2 24.6 -> 27.0 us).
    if (whole && (ncol < 9 ? most : nine_tenths)) return prec == BRI_F64 && ncol == 1 && tiles <= 512;
    // Both whole lines, the cut tiles' runs at least eight sites: the idle lanes cost (8x4x40x64 FP64 x 2 220 -> 343
    // us, 4x8x40x14 bfloat16 links x 7 98 -> 146), except where
    if (whole && run >= 8) {
        if (ncol == 1 && prec != BRI_F32_BF16W) {
            // - large lattices at one right-hand side gain the columns' order (8x28x28x28 FP64 1.21 times);
            if (cut >= 512 && three_quarters) return false;
            // - FP64 takes no further block a CU (4x18x32x8 54 -> 42 us; 4x8x20x24, one more, 25.0 -> 34.5);
            if (prec == BRI_F64) return (tiles + CUS - 1) / CUS > (cut + CUS - 1) / CUS;
            // - the runs are no longer (4x18x20x24 FP32 61 -> 46 us).
            return run > 8;
        }
        // - a batch gets a block a CU or less (FP64 8x6x8x6 x 4 1.3 times), or is one of three, whose cut tiles
        //   carry all three per thread (4x12x28x6 61 -> 43 us);
        if (prec == BRI_F64 && (launch_blocks(tiles, ncol, line) <= CUS || (ncol == 3 && three_quarters))) return false;
        // - the runs are no longer and few lanes idle (4x14x14x64 bfloat16 links x 8 1.3 times).
        return run > 8 || !three_quarters;
    }
    return false;
}

// Replaces the tile configuration by the small-lattice kernel or whole-line tiles where they measured
// faster.
static void lines_default(const Geom &g, int prec, int ncol, int kind, StencilConfig &c) {
    // Up to about a block per CU (two in FP64 batches, six in FP32 and with bfloat16 links) of the small-
    // lattice kernel, eight waves each up to 256 blocks: 8^4 FP64 21.6 -> 10.6 us, FP32 16.7 -> 6.9,
    // bfloat16 links 14.3 -> 6.8; 4^4 x 4 FP64 33.7 -> 8.0.  Beyond, its blocks queue and the tile
    // kernels' shared loads win: FP64 8x8x8x16 24.0 against 22.5 us, 8^4 x 3 35 against 29; FP32
    // 8x8x8x16 x 6 51 against 39, 12^4 x 2 48 against 46.
    const long long blocks16 = (long long)g.V / 16 * ncol;
    if (kind == KERN_BRI && g.V <= SMALL_MAX_SITES && blocks16 <= (prec != BRI_F64 ? 1536 : ncol > 1 ? 512 : 256)) {
        c.small = blocks16 <= 256 ? 8 : 4;
        c.xcd_remap = 1;
        return;
    }
    if (kind == KERN_BRI && rows_fit(g, prec, ncol)) {
        c = StencilConfig{};
        c.nsplit = 4;
        c.xcd_remap = 1;
        c.rows = 48 / g.L[0];
        line_columns(g, c.rows, 36, c);
        return;
    }
    StencilConfig line = c;
    if (!lines_fit(g, &line.lines)) return;
    line.xcd_remap = 1;
    const int tiles = line_tiles(g, line.lines);
    if (kind == KERN_WIL) {
        // Up to 2048 tiles of 16 x 4 stay (16^3x32 FP64 29.9 against 31.7 us, 16^4 FP32 9.7 against 10.4).
        if ((c.colz > 0 && g.V / 64 <= 2048) || cut_stays(g, prec, ncol, kind, c, line)) return;
        // the four one-hop slabs: 960 bytes of FP64 links and spinors a site, deep columns.  32^3x64
        // FP64 755 -> 496 us, FP32 393 -> 312; 24^3x48 FP64 177 -> 166
        if (ncol == 1) {
            line.rpt = 0;
            line.nsplit = g.V / 64 >= 8192 ? 2 : 4;
        }
        line_columns(g, line.lines, 64, line);
        c = line;
        return;
    }
    if (ncol != 2 && xline_fits(g)) return;  // whole-line tiles already
    line.rpt = 0;
    if (prec == BRI_F64 && ncol == 1 && tiles <= CUS / 2) {
        // at most half as many tiles as CUs: twelve waves on each (40 slabs in 4 turns instead of 10), 48x8x4x4
        // 25.0 -> 21.9 us (four waves 23.5), 12x4x8x16 32 -> 21 (22.8); at 192 tiles slower than four
        // (16x16x24x2 26.5 against 25.4), and on cut tiles throughout (2x6x32x12 35.9 against 33.3)
        line.variant = VAR_STANDARD;
        line.nsplit = 12;
        line_columns(g, line.lines, 36, line);
        c = line;
        return;
    }
    // Pairs of right-hand sides pay where at most one place in six is empty: on more than 1024 tiles in FP64 they
    // are level with one per thread for 5, 5% faster for 7 and 12% slower for 3.
    const int pairs = (ncol + 1) / 2;
    const bool paired = ncol > 1 && 6 * ncol >= 10 * pairs;
    // (16 x 4 tiles in columns one row wide: 16^4 overlap apply 4.02 ms, 4.15 in columns of 4 rows; the
    // gradient's batches of 2 and 32 likewise, 13.3 against 13.5 ms; 3 right-hand sides gain, 312 -> 280 us)
    if (prec == BRI_F64 && tiles <= 1024 && c.colz > 0 && (ncol == 1 || paired)) return;
    // One right-hand side per thread on the x-line kernel, or two (FP64) or three per thread on the
    // standard kernel, which loads a link once for them but each neighbour spinor separately.  12
    // right-hand sides at 24^3x48: FP64 12.5 ms (x-line) against 11.0 (R = 2), FP32 6.92 against
    // 6.83 (R = 3); 3 right-hand sides at 20x12x28x24: FP64 705 us (x-line) against 772, FP32 374
    // against 424.
    // Launches of up to a few rounds of blocks take the standard kernel with one per thread: the pairs' blocks are
    // fewer and longer (FP64 up to 1024 blocks, 48x6x16x6 x 2 99 -> 85 us, 4x32x16x6 x 9 143 -> 124), and against
    // the x-line kernel its turns are shorter, 40 slabs in 10 instead of 27 groups in 7 (FP64 up to 1024 tiles,
    // 12^3x24 91 -> 82 us, 8x16x36x2 x 3 41 -> 38; FP32 up to 512 blocks, 16x40x4x12 33.3 -> 29.6, at 576 40.1
    // against 43.9; bfloat16 links 8x24x12x12 32.1 -> 28.6).
    line.variant = VAR_XLINE;
    line.nsplit = 4;
    if (prec == BRI_F64) {
        if (paired && (long long)tiles * pairs >= 4 * CUS) {
            line.variant = VAR_STANDARD;
            line.rpt = 2;
        } else if (tiles <= 4 * CUS) {
            line.variant = VAR_STANDARD;
        }
    } else if ((long long)tiles * ncol <= 2 * CUS) {
        line.variant = VAR_STANDARD;
    } else if (prec == BRI_F32 && ncol >= 9 && tiles >= 512) {
        line.variant = VAR_STANDARD;
        line.rpt = 3;
    }
    if (cut_stays(g, prec, ncol, kind, c, line)) return;
    line_columns(g, line.lines, ncol > 1 ? 16 : prec == BRI_F64 ? 36 : 72, line);
    c = line;
}

// Every launch leaves one pair of sums per tile; a tile holds at least 32 sites on average, 16 in the
// small-lattice kernel.
int stencil_max_slots(const Geom &g) { return g.V <= SMALL_MAX_SITES ? g.V / 16 : g.V / 32; }

// the configuration a launch uses: the installed one, else the default with whole-line tiles where
// bri_stencil_cfg cannot express them
StencilConfig default_config(const Geom &g, int prec, int ncol, int kind) {
    StencilConfig c;
    if (kind == KERN_BRI && tuned_config(g, prec, ncol, &c)) return c;
    return untuned_config(g, prec, ncol, kind);
}

StencilConfig untuned_config(const Geom &g, int prec, int ncol, int kind) {
    StencilConfig c = tile_config(g, prec, ncol, kind);
    lines_default(g, prec, ncol, kind, c);
    return c;
}

}  // namespace bri

extern "C" {

static int apply_common(const bri_geom *geom, const void *W, int prec, double m0, const void *in, void *out, int nrhs,
                        void *stream, bool dag, int kind) {
    using namespace bri;
    StencilArgs a{};
    int rc = geom_check(geom, &a.g);
    if (rc != BRI_OK) return rc;
    if (!W || !in || !out || nrhs < 1 || nrhs > 65535 || a.g.V % 64) return BRI_EINVAL;
    if (prec != BRI_F64 && prec != BRI_F32 && prec != BRI_F32_BF16W) return BRI_EINVAL;
    const size_t sb = (size_t)12 * a.g.V * nrhs * (prec == BRI_F64 ? 16 : 8);
    if (ranges_overlap(in, sb, out, sb)) return BRI_EINVAL;  // neighbours are read while out is written
    a.W = W;
    a.in = in;
    a.out = out;
    a.ncol = nrhs;
    a.kind = kind;
    a.diag = kernel_diag(kind) + m0;
    return stencil_launch(a, prec, dag, EPI_PLAIN, default_config(a.g, prec, nrhs, kind), (hipStream_t)stream);
}

int bri_apply(const bri_geom *geom, const void *W, int prec, double m0, const void *in, void *out, int nrhs,
              void *stream) {
    return apply_common(geom, W, prec, m0, in, out, nrhs, stream, false, bri::KERN_BRI);
}

int bri_apply_dag(const bri_geom *geom, const void *W, int prec, double m0, const void *in, void *out, int nrhs,
                  void *stream) {
    return apply_common(geom, W, prec, m0, in, out, nrhs, stream, true, bri::KERN_BRI);
}

int wil_apply(const bri_geom *geom, const void *W, int prec, double m0, const void *in, void *out, int nrhs,
              void *stream) {
    return apply_common(geom, W, prec, m0, in, out, nrhs, stream, false, bri::KERN_WIL);
}

int wil_apply_dag(const bri_geom *geom, const void *W, int prec, double m0, const void *in, void *out, int nrhs,
                  void *stream) {
    return apply_common(geom, W, prec, m0, in, out, nrhs, stream, true, bri::KERN_WIL);
}

}  // extern "C"

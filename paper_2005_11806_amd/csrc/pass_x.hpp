// x-direction passes of the eigenexpansion solve (Sec. 3.3.1) as block-level
// tile functions, shared by the per-pass kernels and the persistent batch
// kernel:
//  * forward: right-hand-side assembly (Method I, Eq. poisson_me1, a scaled
//    copy, or a refinement residual) fused with the real FFT along x; the
//    half spectrum goes to layout A [k][m][j];
//  * inverse: real inverse FFT along x from layout A and the store of p.
// A tile is `lb` consecutive x-lines (j0 .. j0+lb-1) of one z-plane k; the
// block has 256 threads.
#pragma once

#include <type_traits>

#include "internal.hpp"

namespace psv {

struct XGeom {
    int nx, ny, nz, mx, M, lb, tiles;  // tiles = ny / lb
    int ls;                            // LDS elements from one FFT line to the next
    int stage;                         // forward tile: stencil rows staged in LDS (1) or not (0)
    int win;                           // forward pass: tiles per XCD line window, 0 = plane ranges
    FastDiv by_tiles, by_lb, by_m, by_win;  // division by tiles, lb, M and win
    double inv_dx, inv_dy;
    Radices rad;
};

struct Stencil {
    const double* inv_h;
    const double* inv_g;
    const double* vol;
};

// x-line lengths (nx/2) with a compile-time FFT; others use the runtime one.
// The batched kernels hold those up to 128 of the first list.
#define PSV_X_SIZES(X) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(512)
#define PSV_X_MORE(X) X(8) X(12) X(18) X(36) X(54) X(72) X(108) X(144) X(162) X(384)
// The second list holds further lengths of small and middle size that are in use. In
// neither, and so 1.5 to 3 times slower: odd half-lengths (nx = 6, 18, 54, 162, 486),
// nx of 4, 8 and 12, and 432, 576, 648, 864, 972.
//
// How FP32 transforms round their twiddle products (cmul_sep): a refined or
// iterated result keeps 1e-10 of that rounding. In the second list it is written
// out, the runtime transform's way (which a batch takes for these lengths), and so it
// is in the forward ones of 64 and 512, which would otherwise not round as they did
// in an earlier form of the tile. The rest of the first list is left to the compiler,
// which fuses some stages one way and some the other (neither form written out
// throughout gives the bits of any of them): another compiler may round those
// differently. dir: -1 forward, +1 inverse.
template <typename T>
__host__ __device__ constexpr int x_sep(int M, int dir) {
    if (sizeof(T) == 8) return 0;
    if (M == 64 || M == 512) return dir < 0 ? 2 : 0;
#define PSV_CASE(n) if (M == n) return 0;
    PSV_X_SIZES(PSV_CASE)
#undef PSV_CASE
    return 1;
}
constexpr bool x_compiled(int M) {
    switch (M) {
#define PSV_CASE(n) case n:
        PSV_X_SIZES(PSV_CASE)
        PSV_X_MORE(PSV_CASE)
#undef PSV_CASE
        return true;
        default: return false;
    }
}

// FFT buffers of the x tiles hold lb lines of M elements. Compile-time
// lengths: one pad element after every 8 of a line (Pad8: the radix scatter of
// a Stockham stage then spreads over the LDS banks), and lines x_line_span
// elements apart: the split passes read and write the lb lines of one
// wavenumber from adjacent lanes, 8 lanes (8 x 16 bytes) to an LDS cycle, and a
// stride of 8 / lb modulo 8 puts those on different banks (a stride of 144
// elements, 4 lines: 16 cycles per read and 32 per write of a wave against 9
// and 13 at 146). Runtime lengths: plain lines, M apart.
__host__ __device__ constexpr int x_line_span(int M, int lb) {
    const int want = lb >= 8 ? 1 : 8 / lb;  // modulo 8
    int s = M + M / 8;
    if (lb > 1)
        while ((s & 7) != (want & 7)) ++s;
    return s;
}

// LDS bytes of the x tiles for complex element size csz, with the compile-time
// (ct) or the runtime transform. Inverse: two FFT buffers and the twiddles
// (runtime: the second buffer is the staged half spectrum). Forward: the
// twiddles, then the staged rows (lb + 2 rows, FP64, of the `fields` stencil
// fields: p and rho, p alone for a residual, none for a copy) and two FFT
// buffers. One of these takes the rows' place once they are used up; in a
// tile whose threads make one step each over it (x_one_step) both do, behind
// a barrier: 27 instead of 36 KiB at 256 x 4 lines, five blocks per CU.
constexpr size_t x_rows_bytes(int M, int lb, bool stage, int fields) {
    return stage ? (size_t)fields * (lb + 2) * 2 * M * sizeof(double) : 0;
}
__host__ __device__ constexpr bool x_one_step(int M, int lb, int nt) { return lb * (M / 2) <= nt; }
// Elements from one line to the next
constexpr int x_span(int M, int lb) { return x_compiled(M) ? x_line_span(M, lb) : M; }
constexpr size_t fwd_x_bytes(int M, int lb, bool stage, size_t csz, int mode, bool ct, int nt = 256) {
    const int fields = mode == FWD_CONST ? 0 : (mode == FWD_RESID ? 1 : 2);
    const size_t rows = x_rows_bytes(M, lb, stage, fields);
    const size_t buf = (size_t)lb * (ct ? x_span(M, lb) : M) * csz;
    const size_t tw = (size_t)(ct ? 1 : 2) * M * csz + 16;
    if (ct && rows && x_one_step(M, lb, nt)) return tw + (rows > 2 * buf ? rows : 2 * buf);
    return tw + buf + (rows > buf ? rows : buf);
}
constexpr size_t inv_x_bytes(int M, int lb, size_t csz, bool ct) {
    if (ct) return ((size_t)2 * lb * x_span(M, lb) + M) * csz;
    return ((size_t)lb * M + (size_t)lb * (M + 1) + 2 * (size_t)M) * csz;
}
inline size_t fwd_x_lds(const XGeom& g, size_t csz, int mode, bool ct) {
    return fwd_x_bytes(g.M, g.lb, g.stage != 0, csz, mode, ct);
}
inline size_t inv_x_lds(const XGeom& g, size_t csz, bool ct) { return inv_x_bytes(g.M, g.lb, csz, ct); }
// Which lines per block are admitted and chosen from: by FP64 tiles (forward with
// staged rows or inverse, whichever is larger) of lines M + M / 8 apart, a figure
// that saved and given shapes are held against. The tiles themselves come to a
// little more or less (their lines' spans against no second set of twiddles);
// x_admitted_fit below checks that whatever is admitted fits a block.
constexpr size_t x_lds_max(int nx, int lb) {
    const size_t M = nx / 2, csz = 16, span = (size_t)lb * M + (size_t)lb * M / 8 + 1;
    const size_t rows = x_rows_bytes(nx / 2, lb, true, 2), buf = span * csz;
    const size_t a = buf + 2 * M * csz + 16 + (rows > buf ? rows : buf);
    const size_t half = (size_t)lb * (M + 1);
    const size_t b = (span + (half > span ? half : span) + 2 * M) * csz;
    return a > b ? a : b;
}
constexpr int MAX_LINES_X = 64;  // lines per block that a shape may ask for
constexpr bool smooth23(int n) {
    while (n % 2 == 0) n /= 2;
    while (n % 3 == 0) n /= 3;
    return n == 1;
}
constexpr bool x_admitted_fit() {
    for (int nx = 4; nx <= 1024; nx += 2) {
        for (int lb = 1; lb <= MAX_LINES_X; ++lb) {  // (a divisor of ny)
            if (!smooth23(nx) || !smooth23(lb) || x_lds_max(nx, lb) > (size_t)LDS_MAX_BLOCK) continue;
            for (int ct = 0; ct <= (x_compiled(nx / 2) ? 1 : 0); ++ct) {  // a batch's tiles may be runtime ones
                if (inv_x_bytes(nx / 2, lb, 16, ct) > (size_t)LDS_MAX_BLOCK) return false;
                for (int mode : {FWD_CONST, FWD_METHOD1, FWD_RESID, FWD_METHOD3})
                    for (int stage = 0; stage <= 1; ++stage)
                        if (fwd_x_bytes(nx / 2, lb, stage, 16, mode, ct) > (size_t)LDS_MAX_BLOCK) return false;
            }
        }
    }
    return true;
}

// (1 - rho0/rho_f) (p_R - p_L) across the face between cells L and R, with
// rho_f = (rho_L + rho_R)/2, i.e. (s - 2 rho0)/s with s = rho_L + rho_R.
__device__ __forceinline__ double bflux(double rl, double rr, double pl, double pr, double two_r0) {
    const double s = rl + rr;
    return (s - two_r0) * rcp_nr1(s) * (pr - pl);
}

// rho_f^-1 (p_R - p_L) across the face between cells L and R,
// rho_f = (rho_L + rho_R)/2.
__device__ __forceinline__ double gflux(double rl, double rr, double pl, double pr) {
    return 2.0 * rcp_nr1(rl + rr) * (pr - pl);
}

// 7-point L p at one cell (flux form in z; zero wall flux).
__device__ __forceinline__ double lap_cell(const double* __restrict__ p, int i, int j, int k,
                                           const XGeom& g, const Stencil& st) {
    const size_t plane = (size_t)g.nx * g.ny;
    const size_t row = (size_t)k * plane + (size_t)j * g.nx;
    const size_t c = row + i;
    const int ie = (i + 1 == g.nx) ? 0 : i + 1;
    const int iw = (i == 0) ? g.nx - 1 : i - 1;
    const int jn = (j + 1 == g.ny) ? 0 : j + 1;
    const int js = (j == 0) ? g.ny - 1 : j - 1;
    const double pc = p[c];
    double acc = ((p[row + ie] - pc) - (pc - p[row + iw])) * (g.inv_dx * g.inv_dx);
    acc += ((p[(size_t)k * plane + (size_t)jn * g.nx + i] - pc) -
            (pc - p[(size_t)k * plane + (size_t)js * g.nx + i])) * (g.inv_dy * g.inv_dy);
    const double ft = (k + 1 < g.nz) ? (p[c + plane] - pc) * st.inv_g[k + 1] : 0.0;
    const double fb = (k > 0) ? (pc - p[c - plane]) * st.inv_g[k] : 0.0;
    return acc + (ft - fb) * st.inv_h[k];
}

// Prologue values of a forward tile: the plane's stencil coefficients and the
// mode's scalars.
struct FwdCtx {
    double rho0, two_r0, mean, sc, omega, idx2, idy2, igt, igb, ih;
    bool const_w, has_p;
    int up, dn;  // planes to the operand above and below
};
template <int MODE>
__device__ __forceinline__ FwdCtx fwd_ctx(const XGeom& g, const Stencil& st, const FwdArgs& a, int k) {
    FwdCtx x;
    x.rho0 = (MODE == FWD_METHOD1) ? *a.rho0 : 0.0;
    x.two_r0 = 2.0 * x.rho0;
    x.mean = (MODE == FWD_RESID || (MODE == FWD_METHOD3 && a.mean)) ? *a.mean : 0.0;
    x.sc = ((MODE == FWD_CONST || MODE == FWD_METHOD3) && a.scale) ? a.scale[k] : 1.0;
    // Method III weights the residual by the cell density; a constant weight
    // (min rho) gives the Method-I iteration in the same pressure form
    x.const_w = MODE == FWD_METHOD3 && a.rho0 != nullptr;
    x.omega = x.const_w ? *a.rho0 : 0.0;
    x.idx2 = g.inv_dx * g.inv_dx;
    x.idy2 = g.inv_dy * g.inv_dy;
    // no flux through a wall: the plane on the other side stands in for the one
    // beyond (nz >= 2) and inv_g is taken as 0, so that the tile has no branches
    // over its z faces. What is multiplied by that 0 is then the flux of the face
    // on the other side, finite wherever the result is (the plane itself would
    // not do: a wall cell of density 0 divides by 0 + 0 there).
    const bool top = k + 1 == g.nz, bottom = k == 0;
    x.up = top ? -1 : 1;
    x.dn = bottom ? -1 : 1;
    x.igt = top ? 0.0 : st.inv_g[k + 1];
    x.igb = bottom ? 0.0 : st.inv_g[k];
    x.ih = st.inv_h[k];
    // Method III without a pressure iterate reads p as 0
    x.has_p = MODE != FWD_METHOD3 || a.pprev != nullptr;
    return x;
}

// Global operands of a pair of cells: f (or r_in) and p, rho on the planes
// k +- 1; for tiles without staged rows also the pair, its y neighbour pairs
// and (unless the adjacent lanes hold them) its two x neighbours.
struct FwdPre {
    double2 f, pc, pn, ps, ptz, pbz, rc, rn, rs, rtz, rbz;
    double pw, pe, rw, re;
};
// In-plane values of a pair: the pair, its y neighbour pairs, its x neighbours.
struct FwdNb {
    double2 pc, pn, ps, rc, rn, rs;
    double pw, pe, rw, re;
};
struct FwdSums {
    double res2 = 0.0, r2 = 0.0, rsum = 0.0, qabs = 0.0;
};

// Right-hand side of one pair (cells 2n, 2n+1) from its operands; west(fe, own)
// gives the flux through the west face (own() evaluates it).
template <int MODE, typename West>
__device__ __forceinline__ double2 fwd_pair(const FwdCtx& x, const FwdPre& q, const FwdNb& b,
                                            FwdSums& sum, West&& west) {
    double2 v;
    const double2 pc = b.pc, ptz = q.ptz, pbz = q.pbz;
    if constexpr (MODE == FWD_CONST) {
        v = double2{q.f.x * x.sc, q.f.y * x.sc};
    } else if constexpr (MODE == FWD_METHOD1) {
        const double2 rc = b.rc, rtz = q.rtz, rbz = q.rbz;
        const double t2 = x.two_r0;
        // x faces: west of 2n, between the pair, east of 2n+1
        const double fm = bflux(rc.x, rc.y, pc.x, pc.y, t2);
        const double fe = bflux(rc.y, b.re, pc.y, b.pe, t2);
        const double fw = west(fe, [&] { return bflux(b.rw, rc.x, b.pw, pc.x, t2); });
        double d0 = (fm - fw) * x.idx2, d1 = (fe - fm) * x.idx2;
        d0 += (bflux(rc.x, b.rn.x, pc.x, b.pn.x, t2) - bflux(b.rs.x, rc.x, b.ps.x, pc.x, t2)) * x.idy2;
        d1 += (bflux(rc.y, b.rn.y, pc.y, b.pn.y, t2) - bflux(b.rs.y, rc.y, b.ps.y, pc.y, t2)) * x.idy2;
        const double t0z = bflux(rc.x, rtz.x, pc.x, ptz.x, t2) * x.igt;
        const double t1z = bflux(rc.y, rtz.y, pc.y, ptz.y, t2) * x.igt;
        const double b0z = bflux(rbz.x, rc.x, pbz.x, pc.x, t2) * x.igb;
        const double b1z = bflux(rbz.y, rc.y, pbz.y, pc.y, t2) * x.igb;
        d0 += (t0z - b0z) * x.ih;
        d1 += (t1z - b1z) * x.ih;
        v = double2{d0 + x.rho0 * q.f.x, d1 + x.rho0 * q.f.y};
    } else if constexpr (MODE == FWD_METHOD3) {
        // q = f - D(rho_f^-1 G p), r = rho q (cell density, Eq. new_poisson in
        // pressure form)
        const double2 rc = b.rc, rtz = q.rtz, rbz = q.rbz;
        const double fm = gflux(rc.x, rc.y, pc.x, pc.y);
        const double fe = gflux(rc.y, b.re, pc.y, b.pe);
        const double fw = west(fe, [&] { return gflux(b.rw, rc.x, b.pw, pc.x); });
        double d0 = (fm - fw) * x.idx2, d1 = (fe - fm) * x.idx2;
        d0 += (gflux(rc.x, b.rn.x, pc.x, b.pn.x) - gflux(b.rs.x, rc.x, b.ps.x, pc.x)) * x.idy2;
        d1 += (gflux(rc.y, b.rn.y, pc.y, b.pn.y) - gflux(b.rs.y, rc.y, b.ps.y, pc.y)) * x.idy2;
        const double t0z = gflux(rc.x, rtz.x, pc.x, ptz.x) * x.igt;
        const double t1z = gflux(rc.y, rtz.y, pc.y, ptz.y) * x.igt;
        const double b0z = gflux(rbz.x, rc.x, pbz.x, pc.x) * x.igb;
        const double b1z = gflux(rbz.y, rc.y, pbz.y, pc.y) * x.igb;
        d0 += (t0z - b0z) * x.ih;
        d1 += (t1z - b1z) * x.ih;
        const double q0 = (q.f.x * x.sc - x.mean) - d0, q1 = (q.f.y * x.sc - x.mean) - d1;
        sum.qabs += fabs(q0) + fabs(q1);
        v = double2{(x.const_w ? x.omega : rc.x) * q0, (x.const_w ? x.omega : rc.y) * q1};
    } else {  // residual r - mean - L p
        double l0 = ((pc.y - pc.x) - (pc.x - b.pw)) * x.idx2;
        double l1 = ((b.pe - pc.y) - (pc.y - pc.x)) * x.idx2;
        l0 += ((b.pn.x - pc.x) - (pc.x - b.ps.x)) * x.idy2;
        l1 += ((b.pn.y - pc.y) - (pc.y - b.ps.y)) * x.idy2;
        l0 += ((ptz.x - pc.x) * x.igt - (pc.x - pbz.x) * x.igb) * x.ih;
        l1 += ((ptz.y - pc.y) * x.igt - (pc.y - pbz.y) * x.igb) * x.ih;
        const double rp0 = q.f.x - x.mean, rp1 = q.f.y - x.mean;
        v = double2{rp0 - l0, rp1 - l1};
        sum.res2 += v.x * v.x + v.y * v.y;
        sum.r2 += rp0 * rp0 + rp1 * rp1;
    }
    sum.rsum += v.x + v.y;
    return v;
}

// Per-tile partial sums (when requested) at slot b: one value (vol * sum r)
// for CONST/METHOD1, sum |q| apart for METHOD3, two (sum res^2, sum r~^2) for
// RESID.
template <int MODE>
__device__ __forceinline__ void fwd_partials(const FwdArgs& a, const Stencil& st, const FwdSums& sum,
                                             int k, int b, double* red) {
    if (MODE == FWD_METHOD3 && a.partials_abs) {
        const double s1 = block_sum(sum.qabs, red);
        if (threadIdx.x == 0) a.partials_abs[b] = s1;
        __syncthreads();
    }
    if (MODE != FWD_RESID && a.partials) {
        // FP64 volume-weighted sum of the right-hand side (its mean is the
        // compatibility projection; the FP32 spectrum is too coarse for it)
        const double s1 = block_sum(sum.rsum, red);
        if (threadIdx.x == 0) a.partials[b] = s1 * st.vol[k];
    }
    if (MODE == FWD_RESID) {
        const double s1 = block_sum(sum.res2, red);
        __syncthreads();
        const double s2 = block_sum(sum.r2, red);
        if (threadIdx.x == 0) {
            a.partials[2 * b] = s1;
            a.partials[2 * b + 1] = s2;
        }
    }
}

// Line j of a tile's staged rows rr = 0 .. lb + 1 (lines j0 - 1 .. j0 + lb, periodic).
__device__ __forceinline__ int staged_line(const XGeom& g, int j0, int rr) {
    int j = j0 - 1 + rr;
    j += (j < 0) ? g.ny : 0;
    j -= (j >= g.ny) ? g.ny : 0;
    return j;
}

// Forward tile b, compile-time length N = nx/2, NT threads: the packed input
// z_n = r_2n + i r_2n+1 of the half-length transform is assembled one pair of
// cells per step.
//
// STAGE (and the copy, which has no stencil): a thread takes the pairs n and
// n + N/2 of a line, whose sum and difference are (FP64) the transform's first
// radix-2 stage, so that stage costs no LDS pass and no barrier. Every global
// operand of both pairs (f, and p, rho on the planes k +- 1) is loaded into
// registers together, before the rows j0-1 .. j0+lb of p and rho go to LDS by
// direct loads (64-entry chunks, one per wave instruction), so the two
// overlap. Without: one pair at a time with all its neighbours loaded
// directly, where the caches serve the rows that neighbouring tiles share.
// After the remaining stages a thread reads Z_m and Z_(N-m) once and writes
// both bins they determine. Against every stage and the split of each bin
// through LDS, that is 346 instead of 607 vector and 36 instead of 43.5 LDS
// instructions per wave (counters) and 27 KiB at 256 x 4 lines: 250 -> 233 us per
// pass at 256x256x512 FP64 (1.08 GB; without its transform it takes as long, so
// memory bounds it: 210 us with contiguous spectrum stores, 175 without stores),
// 21.2 -> 18.1 at 128^3. Registers (METHOD1): 96 at half-length 128 and 93 to 95 at
// lengths with a factor of 3, five waves per SIMD; 97 to 99 at the other powers of
// two, and 99 to 106 in METHOD3, four.
template <typename TC, typename TS, int MODE, int N, bool STAGE, int NT>
__device__ __forceinline__ void fwd_x_tile_ct(const XGeom& g, const Stencil& st, const FwdArgs& a,
                                              const c2<TC>* __restrict__ tw_g,
                                              c2<TS>* __restrict__ spec, int b, unsigned char* smem,
                                              double* red, bool norm_only) {
    using C = c2<TC>;
    using P = Pad8;
    constexpr int SEP = x_sep<TC>(N, -1);
    constexpr int M = N, nx = 2 * N, H = N / 2;
    const int k = fdiv(b, g.by_tiles);
    const int j0 = (b - k * g.tiles) * g.lb;
    const int lb = g.lb, ls = g.ls;
    constexpr bool RHO = MODE == FWD_METHOD1 || MODE == FWD_METHOD3;
    constexpr bool TWO = MODE == FWD_CONST || STAGE;  // two pairs per thread and step
    // FP32 keeps radix_list's order: the iterated FP32 solves carry the rounding
    // of their transforms (1e-9 of the gradient at a 1e-10 threshold)
    constexpr bool FIRST2 = TWO && std::is_same<TC, double>::value;
    constexpr int NROW = MODE == FWD_CONST || !STAGE ? 0 : RHO ? 2 : 1;  // staged fields
    C* tw = reinterpret_cast<C*>(smem);  // exp(-2 pi i t / M), t < M
    double2* pt = reinterpret_cast<double2*>(tw + (M + 1) / 2 * 2);  // staged p rows
    double2* rt = pt + (lb + 2) * M;                                 // staged rho rows
    const bool one_step = NROW > 0 && x_one_step(M, lb, NT);
    C* buf1 = reinterpret_cast<C*>(pt);
    C* buf0 = buf1 + lb * ls;
    if (NROW > 0 && !one_step) {
        const int rows = NROW * (lb + 2) * M * (int)(sizeof(double2) / sizeof(C));
        buf0 = buf1 + (rows > lb * ls ? rows : lb * ls);
    }
    const FwdCtx x = fwd_ctx<MODE>(g, st, a, k);
    FwdSums sum;
    const double2* fg = reinterpret_cast<const double2*>(MODE == FWD_RESID ? a.r_in : a.f);
    const double2* pg = reinterpret_cast<const double2*>(a.pprev);
    const double2* rg = reinterpret_cast<const double2*>(a.rho);
    const unsigned plane = (unsigned)M * (unsigned)g.ny;
    // the tile's first pair; a pair of the tile is an offset c from it
    const size_t base = (size_t)k * plane + (size_t)j0 * M;
    const double2 *ft = fg + base, *pk = pg + base, *rk = rg + base;
    const ptrdiff_t upo = (ptrdiff_t)plane * x.up, dno = (ptrdiff_t)plane * x.dn;
    const double2 *pup = pk + upo, *pdn = pk - dno, *rup = rk + upo, *rdn = rk - dno;
    auto z_operands = [&](FwdPre& q, unsigned c) {
        q.f = at_off(ft, c);
        q.ptz = q.pbz = double2{0.0, 0.0};
        if constexpr (MODE != FWD_CONST) {
            if (x.has_p) {
                q.ptz = at_off(pup, c);
                q.pbz = at_off(pdn, c);
            }
            if constexpr (RHO) {
                q.rtz = at_off(rup, c);
                q.rbz = at_off(rdn, c);
            }
        }
    };
    const int lane = (int)threadIdx.x & 63;
    // twiddles: every second entry of the table of exp(-2 pi i t / nx)
    constexpr int TWP = (M + NT - 1) / NT;
    C twr[TWP];
#pragma unroll
    for (int i = 0; i < TWP; ++i) {
        const int t = (int)threadIdx.x + NT * i;
        twr[i] = tw_g[2 * (t < M ? t : 0)];
    }
    auto put_twiddles = [&] {
#pragma unroll
        for (int i = 0; i < TWP; ++i) {
            const int t = (int)threadIdx.x + NT * i;
            if (t < M) tw[t] = twr[i];
        }
    };
    if constexpr (TWO) {
        const int ntask = lb * H;  // pairs n, n + H of line t / H
        FwdPre q0, q1;
        auto prefetch = [&](int t) {
            const unsigned c = (unsigned)(t / H) * M + (unsigned)(t % H);
            z_operands(q0, c);
            z_operands(q1, c + H);
        };
        if ((int)threadIdx.x < ntask) prefetch((int)threadIdx.x);
        if constexpr (MODE != FWD_CONST) {
            constexpr int CPR = (M + 63) / 64;  // chunks per row
            const int prow = x.has_p ? lb + 2 : 0;
            const int nch = (prow + (RHO ? lb + 2 : 0)) * CPR;
            // the chunk arithmetic is the same on every lane of a wave: scalar
            const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
            for (int c = wave; c < nch; c += NT / 64) {
                const int row = c / CPR, part = c - row * CPR;
                const bool rho_row = row >= prow;
                const int rr = rho_row ? row - prow : row;
                const double2* src = (rho_row ? rg : pg) + (size_t)k * plane +
                                     (size_t)(staged_line(g, j0, rr) * M + part * 64);
                double2* dst = (rho_row ? rt : pt) + rr * M + part * 64;
                if (M % 64 == 0 || part * 64 + lane < M) lds_dma16(src + lane, dst);
            }
            if (!x.has_p)
                for (int t = threadIdx.x; t < (lb + 2) * M; t += NT) pt[t] = double2{0.0, 0.0};
        }
        put_twiddles();
        if constexpr (MODE != FWD_CONST) lds_dma_wait();
        __syncthreads();
        // in-plane neighbours of pair n from the staged rows
        auto rows = [&](FwdNb& v, int line, int n) {
            if constexpr (MODE != FWD_CONST) {
                const int o = (line + 1) * M + n;
                const int w = n == 0 ? M - 1 : -1, e = n + 1 == M ? 1 - M : 1;
                v.pc = pt[o];
                v.pn = pt[o + M];
                v.ps = pt[o - M];
                v.pw = pt[o + w].y;
                v.pe = pt[o + e].x;
                if constexpr (RHO) {
                    v.rc = rt[o];
                    v.rn = rt[o + M];
                    v.rs = rt[o - M];
                    v.rw = rt[o + w].y;
                    v.re = rt[o + e].x;
                }
            }
        };
        auto own = [](double, auto f) { return f(); };
        auto step = [&](int t, C& z0, C& z1) {
            const int line = t / H, n = t % H;
            const unsigned c = (unsigned)line * M + (unsigned)n;
            FwdNb v;
            rows(v, line, n);
            const double2 a0 = fwd_pair<MODE>(x, q0, v, sum, own);
            __builtin_amdgcn_sched_barrier(0);  // one pair's operands at a time
            rows(v, line, n + H);
            const double2 a1 = fwd_pair<MODE>(x, q1, v, sum, own);
            if (a.r_out) {
                double2* ro = reinterpret_cast<double2*>(a.r_out) + base;
                at_off(ro, c) = a0;
                at_off(ro, c + H) = a1;
            }
            z0 = C{(TC)a0.x, (TC)a0.y};
            z1 = C{(TC)a1.x, (TC)a1.y};
        };
        // FP64: the first stage, outputs 2n and 2n + 1 of the line
        auto stage0 = [&](int t, C z0, C z1) {
            C* o = buf0 + t / H * ls;
            if constexpr (FIRST2) {
                o += P::at(2 * (t % H));
                o[0] = cadd(z0, z1);
                o[1] = csub(z0, z1);
            } else {
                o[P::at(t % H)] = z0;
                o[P::at(t % H + H)] = z1;
            }
        };
        for (int t0 = 0; t0 < ntask; t0 += NT) {
            const int t = t0 + (int)threadIdx.x;
            C z0, z1;
            if (t < ntask) {
                if (t0) prefetch(t);
                step(t, z0, z1);
            }
            if (one_step) __syncthreads();  // the rows are used up
            if (t < ntask) stage0(t, z0, z1);
        }
    } else {
        // x neighbours of a pair (cell 2n-1 is the .y of pair n-1, cell 2n+2 the
        // .x of pair n+1) from the adjacent lanes where a wave holds whole
        // lines (N divides 64: groups of N lanes, wrapping) or 64 consecutive
        // pairs of one line (64 divides N: only a wave's first and last lanes
        // load theirs). The west face of a pair is the east face of the pair
        // before it (same operands in the same order), so it comes from there.
        constexpr bool XLANE = 64 % N == 0 || N % 64 == 0;
        constexpr int XG = N < 64 ? N : 64;  // lanes per exchange group
        const double* pd = reinterpret_cast<const double*>(pk);
        const double* rd = reinterpret_cast<const double*>(rk);
        const double2 *pp = pg + (size_t)k * plane, *rp = rg + (size_t)k * plane;
        const int npair = lb * M;
        put_twiddles();
        const int g0 = lane & ~(XG - 1), li = lane & (XG - 1);
        const int src_w = g0 + ((li + XG - 1) & (XG - 1)), src_e = g0 + ((li + 1) & (XG - 1));
        for (int t = threadIdx.x; t < npair; t += NT) {
            const int line = t / M, n = t % M, j = j0 + line;
            const unsigned c = (unsigned)t;
            FwdPre q;
            z_operands(q, c);
            // neighbours, as offsets in the plane (rows) and in the tile (x)
            const unsigned cp = (unsigned)(j * M + n);
            const unsigned cn = (j + 1 == g.ny) ? (unsigned)n : cp + M;
            const unsigned cs = (j == 0) ? (unsigned)((g.ny - 1) * M + n) : cp - M;
            const unsigned xw = (unsigned)(2 * t + (n == 0 ? nx - 1 : -1));
            const unsigned xe = (unsigned)(2 * t + (n + 1 == M ? 2 - nx : 2));
            const bool ld_w = !XLANE || (N > 64 && lane == 0);
            const bool ld_e = !XLANE || (N > 64 && lane == 63);
            FwdNb v;
            v.pc = v.pn = v.ps = double2{0.0, 0.0};
            v.pw = v.pe = 0.0;
            if (x.has_p) {
                v.pc = at_off(pk, c);
                v.pn = at_off(pp, cn);
                v.ps = at_off(pp, cs);
                if (ld_w) v.pw = at_off(pd, xw);
                if (ld_e) v.pe = at_off(pd, xe);
            }
            if constexpr (RHO) {
                v.rw = v.re = 1.0;
                v.rc = at_off(rk, c);
                v.rn = at_off(rp, cn);
                v.rs = at_off(rp, cs);
                if (ld_w) v.rw = at_off(rd, xw);
                if (ld_e) v.re = at_off(rd, xe);
            }
            if constexpr (XLANE) {
                auto nb = [&](const double2& cc, double& w, double& e) {
                    const double wl = __shfl(cc.y, src_w, 64), el = __shfl(cc.x, src_e, 64);
                    w = (N > 64 && lane == 0) ? w : wl;
                    e = (N > 64 && lane == 63) ? e : el;
                };
                nb(v.pc, v.pw, v.pe);
                if constexpr (RHO) nb(v.rc, v.rw, v.re);
            }
            const double2 r = fwd_pair<MODE>(x, q, v, sum, [&](double fe, auto own) -> double {
                if constexpr (XLANE) {
                    const double w = __shfl(fe, src_w, 64);
                    if constexpr (N > 64) return lane == 0 ? own() : w;
                    return w;
                } else {
                    return own();
                }
            });
            if (a.r_out) at_off(reinterpret_cast<double2*>(a.r_out) + base, c) = r;
            buf0[line * ls + P::at(n)] = C{(TC)r.x, (TC)r.y};
        }
    }
    // twiddles of the split, in flight during the transform
    const int ntask = lb * H;
    auto task_m = [&](int t) { return fdiv(t, g.by_lb); };
    C ws = tw_g[(int)threadIdx.x < ntask ? task_m((int)threadIdx.x) : 0];
    fwd_partials<MODE>(a, st, sum, k, b, red);
    if (MODE == FWD_RESID && norm_only) return;
    __syncthreads();
    C* Z;
    if constexpr (FIRST2)
        Z = line_stages<N, AfterRadix2<N>, 0, AfterRadix2<N>::list.count, 2, -1, NT, SEP, P>(buf0, buf1, lb, ls, tw);
    else
        Z = line_stages<N, AllRadices<N>, 0, AllRadices<N>::list.count, 1, -1, NT, SEP, P>(buf0, buf1, lb, ls, tw);
    // Split the half-length transform into the real-input spectrum:
    //   E_m = (Z_m + conj Z_{M-m}) / 2, O_m = (Z_m - conj Z_{M-m}) / (2i),
    //   X_m = E_m + w_m O_m, X_{M-m} = conj(E_m - w_m O_m), w_m = exp(-2 pi i m / nx),
    // for m = 1 .. M/2 - 1; task m = 0 writes X_0 = Re Z_0 + Im Z_0,
    // X_M = Re Z_0 - Im Z_0 and X_{M/2} = conj(Z_{M/2}). Lines run fastest, so
    // the lb bins of one m are contiguous in the spectrum.
    c2<TS>* sk = spec + (size_t)k * ((size_t)g.mx * g.ny) + j0;
    for (int t = threadIdx.x; t < ntask; t += NT) {
        const int m = task_m(t), line = t - m * lb;
        if (t != (int)threadIdx.x) ws = tw_g[m];
        const C* zl = Z + line * ls;
        const C zm = zl[P::at(m)];
        const C zc = zl[P::at(m == 0 ? H : M - m)];
        C x0, x1;
        if (m == 0) {
            x0 = C{zm.x + zm.y, (TC)0};
            x1 = C{zm.x - zm.y, (TC)0};
            at_off(sk, (unsigned)(H * g.ny + line)) = cconv<c2<TS>>(cconj(zc));
        } else {
            const C e = C{(TC)0.5 * (zm.x + zc.x), (TC)0.5 * (zm.y - zc.y)};
            const C o = C{(TC)0.5 * (zm.y + zc.y), (TC)-0.5 * (zm.x - zc.x)};
            const C wo = cmul_sep<SEP == 1>(o, ws);
            x0 = cadd(e, wo);
            x1 = cconj(csub(e, wo));
        }
        at_off(sk, (unsigned)(m * g.ny + line)) = cconv<c2<TS>>(x0);
        at_off(sk, (unsigned)((M - m) * g.ny + line)) = cconv<c2<TS>>(x1);
    }
}

// Forward tile b, runtime length.
template <typename TC, typename TS, int MODE, bool STAGE>
__device__ __forceinline__ void fwd_x_tile_rt(const XGeom& g, const Stencil& st, const FwdArgs& a,
                                              const c2<TC>* __restrict__ tw_g,
                                              c2<TS>* __restrict__ spec, int b, unsigned char* smem,
                                              double* red, bool norm_only) {
    using C = c2<TC>;
    const int k = fdiv(b, g.by_tiles);
    const int j0 = (b - k * g.tiles) * g.lb;
    const int M = g.M, nx = 2 * M, lb = g.lb;
    C* buf0 = reinterpret_cast<C*>(smem);
    C* tw = buf0 + lb * M;  // exp(-2 pi i t / nx), t < nx
    // second FFT buffer, 16-byte aligned; with STAGE it first holds the p and
    // rho rows j0-1 .. j0+lb
    const size_t off = ((reinterpret_cast<size_t>(tw + 2 * M) - reinterpret_cast<size_t>(smem)) + 15) & ~size_t(15);
    C* buf1 = reinterpret_cast<C*>(smem + off);
    double2* pt = reinterpret_cast<double2*>(smem + off);
    double2* rt = pt + (lb + 2) * M;
    const unsigned plane = (unsigned)M * (unsigned)g.ny;
    const FwdCtx x = fwd_ctx<MODE>(g, st, a, k);
    FwdSums sum;
    constexpr bool RHO = MODE == FWD_METHOD1 || MODE == FWD_METHOD3;
    constexpr bool ROWS = MODE != FWD_CONST && STAGE;
    constexpr int PF = (MODE == FWD_CONST || STAGE) ? 2 : 1;
    const double* pd = a.pprev;
    const double* rd = a.rho;
    const int npair = lb * M;
    const double2* fg = reinterpret_cast<const double2*>(MODE == FWD_RESID ? a.r_in : a.f);
    const double2* pg = reinterpret_cast<const double2*>(a.pprev);
    const double2* rg = reinterpret_cast<const double2*>(a.rho);
    const unsigned base = (unsigned)k * plane + (unsigned)j0 * M;
    auto prefetch = [&](int t0, FwdPre* pre) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int t = t0 + u * 256;
            FwdPre& q = pre[u];
            q.pc = q.pn = q.ps = q.ptz = q.pbz = double2{0.0, 0.0};
            q.rc = q.rn = q.rs = q.rtz = q.rbz = double2{1.0, 1.0};
            q.pw = q.pe = 0.0;
            q.rw = q.re = 1.0;
            if (t < npair) {
                const unsigned c = base + (unsigned)t;
                q.f = fg[c];
                if (MODE == FWD_CONST) continue;
                const unsigned cu = c + (unsigned)x.up * plane, cd = c - (unsigned)x.dn * plane;
                if (x.has_p) {
                    q.ptz = pg[cu];
                    q.pbz = pg[cd];
                }
                if (RHO) {
                    q.rtz = rg[cu];
                    q.rbz = rg[cd];
                }
                if (!STAGE) {
                    const int line = fdiv(t, g.by_m), n = t - line * M, j = j0 + line;
                    // neighbour pairs in y (periodic) and cells in x (periodic in the line)
                    const unsigned cn = c + (unsigned)((j + 1 == g.ny) ? -(g.ny - 1) * M : M);
                    const unsigned cs = c - (unsigned)((j == 0) ? -(g.ny - 1) * M : M);
                    const unsigned xw = 2 * c + (unsigned)(n == 0 ? nx - 1 : -1);
                    const unsigned xe = 2 * c + (unsigned)(n + 1 == M ? 2 - nx : 2);
                    if (x.has_p) {
                        q.pc = pg[c];
                        q.pn = pg[cn];
                        q.ps = pg[cs];
                        q.pw = pd[xw];
                        q.pe = pd[xe];
                    }
                    if (RHO) {
                        q.rc = rg[c];
                        q.rn = rg[cn];
                        q.rs = rg[cs];
                        q.rw = rd[xw];
                        q.re = rd[xe];
                    }
                }
            }
        }
    };
    FwdPre cur[PF];
    prefetch(threadIdx.x, cur);
    // rows and twiddles to LDS through registers, every load of a thread issued
    // before its LDS writes (a p element and the rho element at the same place
    // share their address)
    {
        const int nst = ROWS ? (lb + 2) * M : 0;
        auto src = [&](int t) {
            const int rr = fdiv(t, g.by_m);
            return (unsigned)k * plane + (unsigned)staged_line(g, j0, rr) * M + (unsigned)(t - rr * M);
        };
        if constexpr (ROWS && RHO) {
            struct PR {
                double2 p, r;
            };
            const double2* pv = x.has_p ? pg : rg;  // a valid array where p is absent
            block_copy<4, PR>(
                nst,
                [&](int t) {
                    const unsigned i = src(t);
                    return PR{pv[i], rg[i]};
                },
                [&](int t, PR v) {
                    pt[t] = x.has_p ? v.p : double2{0.0, 0.0};
                    rt[t] = v.r;
                });
        } else if constexpr (ROWS) {
            block_copy<4, double2>(nst, [&](int t) { return pg[src(t)]; },
                                   [&](int t, double2 v) { pt[t] = v; });
        }
        block_copy<2, C>(2 * M, [&](int t) { return tw_g[t]; }, [&](int t, C v) { tw[t] = v; });
        __syncthreads();
    }
    for (int t0 = threadIdx.x; t0 < npair; t0 += PF * 256) {
        if (t0 != (int)threadIdx.x) prefetch(t0, cur);
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int t = t0 + u * 256;
            if (t >= npair) break;
            const int line = fdiv(t, g.by_m), n = t - line * M;
            const FwdPre& q = cur[u];
            FwdNb v;
            if constexpr (ROWS) {
                const int o = (line + 1) * M + n;
                const int w = n == 0 ? M - 1 : -1, e = n + 1 == M ? 1 - M : 1;
                v.pc = pt[o];
                v.pn = pt[o + M];
                v.ps = pt[o - M];
                v.pw = pt[o + w].y;
                v.pe = pt[o + e].x;
                if constexpr (RHO) {
                    v.rc = rt[o];
                    v.rn = rt[o + M];
                    v.rs = rt[o - M];
                    v.rw = rt[o + w].y;
                    v.re = rt[o + e].x;
                }
            } else if constexpr (MODE != FWD_CONST) {
                v = FwdNb{q.pc, q.pn, q.ps, q.rc, q.rn, q.rs, q.pw, q.pe, q.rw, q.re};
            }
            const double2 r = fwd_pair<MODE>(x, q, v, sum, [](double, auto f) { return f(); });
            if (a.r_out) reinterpret_cast<double2*>(a.r_out)[base + (unsigned)t] = r;
            buf0[t] = C{(TC)r.x, (TC)r.y};
        }
    }
    fwd_partials<MODE>(a, st, sum, k, b, red);
    if (MODE == FWD_RESID && norm_only) return;
    __syncthreads();
    C* Z = lds_fft<-1>(buf0, buf1, M, lb, M, g.rad, tw, 2 * M);
    // Split the half-length transform into the real-input spectrum:
    //   E_m = (Z_m + conj Z_{M-m}) / 2, O_m = (Z_m - conj Z_{M-m}) / (2i),
    //   X_m = E_m + exp(-2 pi i m / nx) O_m, m = 0..M.
    const int nout = (M + 1) * lb;
    c2<TS>* sk = spec + (size_t)k * ((size_t)g.mx * g.ny) + j0;
    for (int t = threadIdx.x; t < nout; t += 256) {
        const int m = fdiv(t, g.by_lb);
        const int line = t - m * lb;
        const C zm = Z[line * M + (m == M ? 0 : m)];
        const C zc = cconj(Z[line * M + (m == 0 ? 0 : M - m)]);
        const C e = C{(TC)0.5 * (zm.x + zc.x), (TC)0.5 * (zm.y + zc.y)};
        const C o = C{(TC)0.5 * (zm.y - zc.y), (TC)-0.5 * (zm.x - zc.x)};
        const C y = cadd(e, cmul(tw[m], o));
        at_off(sk, (unsigned)(m * g.ny + line)) = cconv<c2<TS>>(y);
    }
}

// Forward tile b. N = nx/2 as a compile-time constant, or 0 (runtime length).
// norm_only (RESID): the partial sums alone, without the transform.
template <typename TC, typename TS, int MODE, int N, bool STAGE = true, int NT = 256>
__device__ __forceinline__ void fwd_x_tile(const XGeom& g, const Stencil& st, const FwdArgs& a,
                                           const c2<TC>* __restrict__ tw_g,
                                           c2<TS>* __restrict__ spec, int b, unsigned char* smem,
                                           double* red, bool norm_only = false) {
    if constexpr (N > 0)
        fwd_x_tile_ct<TC, TS, MODE, N, STAGE, NT>(g, st, a, tw_g, spec, b, smem, red, norm_only);
    else
        fwd_x_tile_rt<TC, TS, MODE, STAGE>(g, st, a, tw_g, spec, b, smem, red, norm_only);
}

// One result of an inverse tile (pair index c): p = s x, or p = old + s x.
template <int MODE, typename C>
__device__ __forceinline__ void inv_store(double2* out2, unsigned c, C v, double s, double2 old) {
    double2 x{(double)v.x * s, (double)v.y * s};
    if (MODE == INV_ADD) {
        x.x += old.x;
        x.y += old.y;
    }
    st_stream(&at_off(out2, c), x);
}

// Inverse tile b: p = scale * x (STORE), p += scale * x (ADD) or
// p = scale * vol[k] * x (SCALE). Compile-time length, NT threads: a thread
// loads the bins X_m and X_{M-m} of a line straight into registers (each bin
// once) and forms both inputs they determine of the half-length transform,
//   Z_m = E_m + i O_m, Z_{M-m} = conj(E_m) + i conj(O_m),
//   E_m = (X_m + conj X_{M-m}) / 2, O_m = (X_m - conj X_{M-m}) conj(w_m) / 2,
// w_m = exp(-2 pi i m / nx); task m = 0 takes X_0, X_M (real parts: a real
// field has real DC and Nyquist bins) and Z_{M/2} = conj X_{M/2}. The last
// stage's butterflies store their outputs, neighbouring lanes neighbouring
// pairs, without another pass through LDS. Against bins staged in LDS and every
// stage through it: 128 instead of 224 vector and 14.5 instead of 24.8 LDS
// instructions per wave and step (counters); 103 -> 90 us at 256x256x512 FP64 and 4
// lines, 83 at 8 (540 MB, 6.5 TB/s), 10.7 -> 7.1 at 128^3.
template <typename TC, typename TS, int MODE, int N, int NT>
__device__ __forceinline__ void inv_x_tile_ct(const XGeom& g, const c2<TC>* __restrict__ tw_g,
                                              const c2<TS>* __restrict__ spec,
                                              double* __restrict__ out,
                                              const double* __restrict__ vol, double scale, int b,
                                              unsigned char* smem) {
    using C = c2<TC>;
    using P = Pad8;
    constexpr int SEP = x_sep<TC>(N, 1);
    constexpr int M = N, H = N / 2;
    const int k = fdiv(b, g.by_tiles);
    const int j0 = (b - k * g.tiles) * g.lb;
    const int lb = g.lb, ls = g.ls;
    C* buf0 = reinterpret_cast<C*>(smem);
    C* buf1 = buf0 + lb * ls;
    C* tw = buf1 + lb * ls;  // exp(-2 pi i t / M), t < M
    const c2<TS>* sk = spec + (size_t)k * ((size_t)g.mx * g.ny) + j0;
    const int ntask = lb * H;
    struct Bins {
        C w, xm, xc, xh;
    };
    auto bins = [&](int t) {
        const int m = fdiv(t, g.by_lb), line = t - m * lb;
        Bins q;
        q.w = tw_g[m];
        q.xm = cconv<C>(at_off(sk, (unsigned)(m * g.ny + line)));
        q.xc = cconv<C>(at_off(sk, (unsigned)((M - m) * g.ny + line)));
        q.xh = C{(TC)0, (TC)0};
        if (m == 0) q.xh = cconv<C>(at_off(sk, (unsigned)(H * g.ny + line)));
        return q;
    };
    auto put = [&](int t, const Bins& q) {
        const int m = fdiv(t, g.by_lb), line = t - m * lb;
        C xm = q.xm, xc = q.xc;
        if (m == 0) xm.y = xc.y = (TC)0;
        const C e = C{(TC)0.5 * (xm.x + xc.x), (TC)0.5 * (xm.y - xc.y)};
        const C d = C{(TC)0.5 * (xm.x - xc.x), (TC)0.5 * (xm.y + xc.y)};
        const C o = cmul_sep<SEP>(d, cconj(q.w));
        C* zl = buf0 + line * ls;
        zl[P::at(m)] = C{e.x - o.y, e.y + o.x};
        zl[P::at(m == 0 ? H : M - m)] = m == 0 ? cconj(q.xh) : C{e.x + o.y, o.x - e.y};
    };
    const int tid = (int)threadIdx.x;
    Bins first;
    if (tid < ntask) first = bins(tid);
    // twiddles behind the first bins, outside any branch: there an array of them
    // goes to scratch memory (1024x64x48 step: 100 us, 97 without)
    constexpr int TWP = (M + NT - 1) / NT;
    C twr[TWP];
#pragma unroll
    for (int i = 0; i < TWP; ++i) {
        const int e = tid + NT * i;
        twr[i] = tw_g[2 * (e < M ? e : 0)];
    }
    if (tid < ntask) put(tid, first);
    for (int t = tid + NT; t < ntask; t += NT) put(t, bins(t));
#pragma unroll
    for (int i = 0; i < TWP; ++i) {
        const int e = tid + NT * i;
        if (e < M) tw[e] = twr[i];
    }
    __syncthreads();
    using L = AllRadices<N>;
    constexpr int LAST = L::list.count - 1;
    const C* z = line_stages<N, L, 0, LAST, 1, +1, NT, SEP, P>(buf0, buf1, lb, ls, tw);
    constexpr int R = L::list.r[LAST], NB = N / R;
    const double s = (MODE == INV_SCALE) ? scale * vol[k] : scale;
    double2* out2 = reinterpret_cast<double2*>(out) + ((size_t)k * g.ny + j0) * M;
    for (int t = threadIdx.x; t < lb * NB; t += NT) {
        const int line = t / NB, j = t - line * NB;
        const unsigned c = (unsigned)line * M + (unsigned)j;
        double2 old[R] = {};
        if (MODE == INV_ADD) {
#pragma unroll
            for (int r = 0; r < R; ++r) old[r] = at_off(out2, c + r * NB);
        }
        C v[R];
        stockham_load_ct<R, +1, NB, NB, 1, SEP, P>(z + line * ls, j, tw, v);
#pragma unroll
        for (int r = 0; r < R; ++r) inv_store<MODE>(out2, c + r * NB, v[r], s, old[r]);
    }
}

// The same for a runtime length, through LDS.
template <typename TC, typename TS, int MODE>
__device__ __forceinline__ void inv_x_tile_rt(const XGeom& g, const c2<TC>* __restrict__ tw_g,
                                              const c2<TS>* __restrict__ spec,
                                              double* __restrict__ out,
                                              const double* __restrict__ vol, double scale, int b,
                                              unsigned char* smem) {
    using C = c2<TC>;
    const int k = fdiv(b, g.by_tiles);
    const int j0 = (b - k * g.tiles) * g.lb;
    const int M = g.M, lb = g.lb;
    C* buf0 = reinterpret_cast<C*>(smem);
    C* xb = buf0 + lb * M;        // lb x (M+1), later the FFT's second buffer
    C* tw = xb + lb * (M + 1);    // exp(-2 pi i t / nx), t < nx
    const c2<TS>* sk = spec + (size_t)k * ((size_t)g.mx * g.ny) + j0;
    const int nin = (M + 1) * lb;
    // one index space: the lb lines' M + 1 bins, then the 2 M twiddles
    block_copy<4, C>(
        nin + 2 * M,
        [&](int t) {
            const int m = fdiv(t, g.by_lb);
            return t < nin ? cconv<C>(sk[(unsigned)m * (unsigned)g.ny + (unsigned)(t - m * lb)]) : tw_g[t - nin];
        },
        [&](int t, C x) {
            if (t < nin) {
                const int m = fdiv(t, g.by_lb);
                if (m == 0 || m == M) x.y = (TC)0;  // a real field has real DC and Nyquist bins
                xb[(t - m * lb) * (M + 1) + m] = x;
            } else {
                tw[t - nin] = x;
            }
        });
    __syncthreads();
    for (int t = threadIdx.x; t < M * lb; t += 256) {
        const int line = fdiv(t, g.by_m);
        const int m = t - line * M;
        const C xm = xb[line * (M + 1) + m];
        const C xc = cconj(xb[line * (M + 1) + (M - m)]);
        const C e = C{(TC)0.5 * (xm.x + xc.x), (TC)0.5 * (xm.y + xc.y)};
        const C d = C{(TC)0.5 * (xm.x - xc.x), (TC)0.5 * (xm.y - xc.y)};
        const C o = cmul(d, cconj(tw[m]));
        buf0[t] = C{e.x - o.y, e.y + o.x};
    }
    __syncthreads();
    C* z = lds_fft<+1>(buf0, xb, M, lb, M, g.rad, tw, 2 * M);
    const double s = (MODE == INV_SCALE) ? scale * vol[k] : scale;
    double2* out2 = reinterpret_cast<double2*>(out) + ((size_t)k * g.ny + j0) * M;
    for (int t = threadIdx.x; t < lb * M; t += 256)
        inv_store<MODE>(out2, (unsigned)t, z[t], s,
                        MODE == INV_ADD ? at_off(out2, (unsigned)t) : double2{0.0, 0.0});
}

template <typename TC, typename TS, int MODE, int N, int NT = 256>
__device__ __forceinline__ void inv_x_tile(const XGeom& g, const c2<TC>* __restrict__ tw_g,
                                           const c2<TS>* __restrict__ spec,
                                           double* __restrict__ out,
                                           const double* __restrict__ vol, double scale, int b,
                                           unsigned char* smem) {
    if constexpr (N > 0)
        inv_x_tile_ct<TC, TS, MODE, N, NT>(g, tw_g, spec, out, vol, scale, b, smem);
    else
        inv_x_tile_rt<TC, TS, MODE>(g, tw_g, spec, out, vol, scale, b, smem);
}

// Geometry of the x tiles; `inverse` selects the inverse pass's lines per block.
inline XGeom make_xgeom(const Plan& p, bool inverse = false) {
    XGeom g;
    g.nx = p.nx;
    g.ny = p.ny;
    g.nz = p.nz;
    g.mx = p.mx;
    g.M = p.nx / 2;
    g.lb = inverse ? p.lp.lbx_inv : p.lp.lbx;
    g.tiles = p.ny / g.lb;
    g.ls = x_span(g.M, g.lb);
    g.by_tiles = fast_div(g.tiles);
    g.by_lb = fast_div(g.lb);
    g.by_m = fast_div(g.M);
    g.stage = p.lp.xstage;
    g.win = (!inverse && p.lp.xorder && g.tiles % 8 == 0) ? g.tiles / 8 : 0;
    g.by_win = fast_div(g.win > 1 ? g.win : 1);
    g.inv_dx = 1.0 / p.dx;
    g.inv_dy = 1.0 / p.dy;
    g.rad = p.rad_xh;
    return g;
}

}  // namespace psv

// Device side of the batched solves: problem descriptors and one tile of one
// pass of one problem, from the same block-level tile functions as the single
// solve (pass_x.hpp, pass_yz.hpp). Included by the translation units that
// instantiate the per-pass and the persistent kernels per precision.
#pragma once

#include <algorithm>
#include <cstring>
#include <vector>

#include "pass_x.hpp"
#include "pass_yz.hpp"

namespace psv {

enum BKind : int {
    K_MINP = 0,  // partial min(rho) with first index
    K_MINF,      // rho0: given value or the reduced minimum
    K_FWD,       // assembly + forward x (CONST or METHOD1)
    K_MEAN,      // FP64 volume-weighted mean of the RHS from the forward partials (mixed)
    K_Y,         // forward y + chunk elimination of the z solve
    K_Z,         // z interface systems + zero mode (mean to S_RHS_MEAN)
    K_Z2,        // same, mean discarded (refinement corrections)
    K_YI,        // z back substitution + inverse y
    K_INV,       // inverse x, store
    K_INVADD,    // inverse x, accumulate
    K_RES,       // fused residual + forward x (refinement)
    K_NRM,       // relres from the residual partials; set done when <= tol
    K_CHK,       // standalone residual (final check)
    K_CHKF,      // relres of the final check
    K_NKIND
};

// cells per min tile: small enough that a problem of 128^3 fills the GPU with
// 256 of them (65536 left 408 blocks for 16 problems, 27 million cells, with one
// load in flight per thread: 128 us)
constexpr int MIN_TILE = 8192;
constexpr int RES_TILE = 2048;   // cells per residual tile
constexpr int MAX_MIN_TILES = 256;

struct ProblemDesc {
    XGeom xg;   // forward x tiles (the plan's lines per block and stencil variant)
    XGeom xgi;  // inverse x tiles (the plan's own lines per block)
    Stencil st;
    ZArgs z;  // rhs_mean set per kind at run time
    int method, fp32;
    Radices rad_y;
    const void* twx;
    const void* twy;
    void* spec;
    double* r_ws;
    double* partials;
    double* scal;
    int* flags;
    double tol;
    double vtotal;  // total volume
    size_t ncell;
    int ntiles[K_NKIND];
};

struct ProblemIO {
    const double* f;
    const double* rho;
    const double* pprev;
    double* pout;
    double rho0;  // <= 0: min(rho)
    int want_r;   // store the FP64 RHS (refinement or final check)
};

inline int kind_tiles(const Plan& p, int kind) {
    switch (kind) {
        case K_MINP: return std::min<int>(MAX_MIN_TILES, (int)((p.ncell() + MIN_TILE - 1) / MIN_TILE));
        case K_FWD: case K_RES: return fwd_x_blocks(p);
        case K_INV: case K_INVADD: return (p.ny / p.lp.lbx_inv) * p.nz;
        case K_Y: case K_YI: return yz_tiles(p);
        case K_Z: case K_Z2: return ifc_tiles(p);
        case K_CHK: return (int)((p.ncell() + RES_TILE - 1) / RES_TILE);
        default: return 1;
    }
}

// ---------------------------------------------------------------------------
// device: small tiles
__device__ void minp_tile(const ProblemDesc& D, const ProblemIO& io, int b) {
    __shared__ double sv[4];
    __shared__ int si[4];
    const int nt = D.ntiles[K_MINP];
    const size_t n2 = D.ncell / 2, chunk = (n2 + nt - 1) / nt;  // pairs (nx is even)
    const size_t c0 = (size_t)b * chunk;
    double best = __builtin_inf();
    int bi = 0x7fffffff;
    min_share(reinterpret_cast<const double2*>(io.rho), c0, min(n2, c0 + chunk), best, bi);
    block_argmin(best, bi, sv, si);
    if (threadIdx.x == 0) {
        D.partials[b] = best;
        D.partials[MAX_MIN_TILES + b] = (double)bi;
    }
}

__device__ void minf_tile(const ProblemDesc& D, const ProblemIO& io) {
    __shared__ double sv[4];
    __shared__ int si[4];
    if (io.rho0 > 0.0) {
        if (threadIdx.x == 0) D.scal[S_RHO0] = io.rho0;
        return;
    }
    double best = __builtin_inf();
    int bi = 0x7fffffff;
    if ((int)threadIdx.x < D.ntiles[K_MINP])  // at most MAX_MIN_TILES = 256
        argmin_merge(best, bi, D.partials[threadIdx.x], (int)D.partials[MAX_MIN_TILES + threadIdx.x]);
    block_argmin(best, bi, sv, si);
    if (threadIdx.x == 0) {
        D.scal[S_RHO0] = best;
        D.flags[F_ARGMIN] = bi;
    }
}

// sum of `per` interleaved partials over nb tiles, on thread 0
__device__ double sum_partials(const double* p, int nb, int per, int q, double* red) {
    return block_sum(thread_share(p, nb, per, q), red);
}

__device__ void mean_tile(const ProblemDesc& D, double* red) {
    const double s = sum_partials(D.partials, D.ntiles[K_FWD], 1, 0, red);
    if (threadIdx.x == 0) D.scal[S_RHS_MEAN] = s / D.vtotal;
}

__device__ void nrm_tile(const ProblemDesc& D, int ntiles, double* red, bool set_done) {
    const double2 ab = thread_share2(D.partials, ntiles);
    const double a = block_sum(ab.x, red);
    __syncthreads();
    const double b = block_sum(ab.y, red);
    if (threadIdx.x == 0) {
        const double rr = b > 0.0 ? sqrt(a / b) : 0.0;
        D.scal[S_RELRES] = rr;
        if (set_done && rr <= D.tol) D.flags[F_DONE] = 1;
        if (set_done) D.flags[F_STEPS] += (rr <= D.tol) ? 0 : 1;
    }
}

__device__ void chk_tile(const ProblemDesc& D, const ProblemIO& io, int b, double* red) {
    const XGeom& g = D.xg;
    const double mean = D.scal[S_RHS_MEAN];
    const size_t c0 = (size_t)b * RES_TILE;
    double s1 = 0.0, s2 = 0.0;
    for (int t = threadIdx.x; t < RES_TILE; t += 256) {
        const size_t c = c0 + t;
        if (c >= D.ncell) break;
        const int i = (int)(c % g.nx);
        const size_t q = c / g.nx;
        const int j = (int)(q % g.ny);
        const int k = (int)(q / g.ny);
        const double rp = D.r_ws[c] - mean;
        const double res = rp - lap_cell(io.pout, i, j, k, g, D.st);
        s1 += res * res;
        s2 += rp * rp;
    }
    const double a = block_sum(s1, red);
    __syncthreads();
    const double bb = block_sum(s2, red);
    if (threadIdx.x == 0) {
        D.partials[2 * b] = a;
        D.partials[2 * b + 1] = bb;
    }
}

// ---------------------------------------------------------------------------
// device: one tile of one pass of one problem
#define PSV_BX_SIZES(X) X(16) X(24) X(32) X(48) X(64) X(96) X(128)
inline bool bx_compiled(int M) {
    switch (M) {
#define PSV_CASE(n) case n:
        PSV_BX_SIZES(PSV_CASE)
#undef PSV_CASE
        return true;
        default: return false;
    }
}

template <typename T, int MODE, bool STAGE>
__device__ __forceinline__ void run_fwd_s(const ProblemDesc& D, const FwdArgs& a, int b,
                                          unsigned char* smem, double* red) {
    const c2<T>* tw = reinterpret_cast<const c2<T>*>(D.twx);
    c2<T>* sp = reinterpret_cast<c2<T>*>(D.spec);
    switch (D.xg.M) {
#define PSV_CASE(n) case n: fwd_x_tile<T, T, MODE, n, STAGE>(D.xg, D.st, a, tw, sp, b, smem, red); return;
        PSV_BX_SIZES(PSV_CASE)
#undef PSV_CASE
        default: fwd_x_tile<T, T, MODE, 0, STAGE>(D.xg, D.st, a, tw, sp, b, smem, red); return;
    }
}

// Forward x tile in the problem's stencil variant: SEL = 1 staged rows, 0
// direct loads (per-pass kernels, one launch per variant), -1 chosen from the
// problem's geometry at run time (persistent kernel). The constant-
// coefficient copy has no stencil and always takes the staged variant.
template <typename T, int MODE, int SEL>
__device__ __forceinline__ void run_fwd(const ProblemDesc& D, const FwdArgs& a, int b,
                                        unsigned char* smem, double* red) {
    if constexpr (MODE == FWD_CONST || SEL == 1) {
        run_fwd_s<T, MODE, true>(D, a, b, smem, red);
    } else if constexpr (SEL == 0) {
        run_fwd_s<T, MODE, false>(D, a, b, smem, red);
    } else {
        if (D.xg.stage)
            run_fwd_s<T, MODE, true>(D, a, b, smem, red);
        else
            run_fwd_s<T, MODE, false>(D, a, b, smem, red);
    }
}

template <typename T, int MODE>
__device__ __forceinline__ void run_inv(const ProblemDesc& D, double* out, int b, unsigned char* smem) {
    const c2<T>* tw = reinterpret_cast<const c2<T>*>(D.twx);
    const c2<T>* sp = reinterpret_cast<const c2<T>*>(D.spec);
    const double sc = 2.0 / ((double)D.xg.nx * D.xg.ny);
    switch (D.xgi.M) {
#define PSV_CASE(n) case n: inv_x_tile<T, T, MODE, n>(D.xgi, tw, sp, out, D.st.vol, sc, b, smem); return;
        PSV_BX_SIZES(PSV_CASE)
#undef PSV_CASE
        default: inv_x_tile<T, T, MODE, 0>(D.xgi, tw, sp, out, D.st.vol, sc, b, smem); return;
    }
}

// KCS: the problem's chunk rows, or -1 (chosen at run time)
template <typename T, bool INV, int N, int KCS>
__device__ __forceinline__ void yz_tile(const ProblemDesc& D, c2<T>* sp, const c2<T>* tw, int b,
                                        unsigned char* smem) {
    auto tile = [&](auto kc) {
        constexpr int KC = decltype(kc)::value;
        if constexpr (INV)
            yz_inv_tile<T, N, KC>(D.z, D.rad_y, sp, tw, b, smem);
        else
            yz_fwd_tile<T, N, KC>(D.z, D.rad_y, sp, tw, b, smem);
    };
    if constexpr (KCS > 0)
        tile(std::integral_constant<int, KCS>{});
    else
        with_kc(D.z.kc, tile);
}

template <typename T, bool INV, int KCS>
__device__ __forceinline__ void run_yz(const ProblemDesc& D, int b, unsigned char* smem) {
    const c2<T>* tw = reinterpret_cast<const c2<T>*>(D.twy);
    c2<T>* sp = reinterpret_cast<c2<T>*>(D.spec);
    switch (D.xg.ny) {
#define PSV_CASE(n) case n: yz_tile<T, INV, n, KCS>(D, sp, tw, b, smem); return;
        PSV_YZ_SIZES(PSV_CASE)
#undef PSV_CASE
        default: yz_tile<T, INV, 0, KCS>(D, sp, tw, b, smem); return;
    }
}

// QM: register rows per lane, at least ifc_qmax of the problem, or -1 (chosen
// at run time)
template <typename T, int QM>
__device__ __forceinline__ void run_ifc(const ProblemDesc& D, double* mean_out, int b,
                                        unsigned char* smem) {
    ZArgs z = D.z;
    z.rhs_mean = mean_out;
    ifc_tile<T, (QM > 0 ? QM : 0)>(z, reinterpret_cast<c2<T>*>(D.spec), b, smem);
}

template <typename T, int KIND, int SEL = -1>
__device__ __forceinline__ void run_task(const ProblemDesc& D, const ProblemIO& io, int b,
                                         unsigned char* smem, double* red) {
    // The done flag is cleared before the first pass and set only by the norm
    // tile of a refinement round, so every tile of a converged problem may
    // return at once.
    if (D.fp32 && D.flags[F_DONE]) return;
    if constexpr (KIND == K_MINP) {
        minp_tile(D, io, b);
    } else if constexpr (KIND == K_MINF) {
        minf_tile(D, io);
    } else if constexpr (KIND == K_FWD) {
        FwdArgs a{};
        a.f = io.f;
        a.rho = io.rho;
        a.pprev = io.pprev;
        a.rho0 = D.scal + S_RHO0;
        a.r_out = io.want_r ? D.r_ws : nullptr;
        a.partials = D.fp32 ? D.partials : nullptr;
        if (D.method == PSV_SPLIT_RHO0) {
            a.mode = FWD_METHOD1;
            run_fwd<T, FWD_METHOD1, SEL>(D, a, b, smem, red);
        } else {
            a.mode = FWD_CONST;
            run_fwd<T, FWD_CONST, SEL>(D, a, b, smem, red);
        }
    } else if constexpr (KIND == K_MEAN) {
        mean_tile(D, red);
    } else if constexpr (KIND == K_Y) {
        run_yz<T, false, SEL>(D, b, smem);
    } else if constexpr (KIND == K_YI) {
        run_yz<T, true, SEL>(D, b, smem);
    } else if constexpr (KIND == K_Z) {
        run_ifc<T, SEL>(D, D.scal + (D.fp32 ? S_MEAN2 : S_RHS_MEAN), b, smem);
    } else if constexpr (KIND == K_Z2) {
        run_ifc<T, SEL>(D, D.scal + S_MEAN2, b, smem);
    } else if constexpr (KIND == K_INV) {
        run_inv<T, INV_STORE>(D, io.pout, b, smem);
    } else if constexpr (KIND == K_INVADD) {
        run_inv<T, INV_ADD>(D, io.pout, b, smem);
    } else if constexpr (KIND == K_RES) {
        FwdArgs a{};
        a.mode = FWD_RESID;
        a.r_in = D.r_ws;
        a.pprev = io.pout;
        a.mean = D.scal + S_RHS_MEAN;
        a.partials = D.partials;
        run_fwd<T, FWD_RESID, SEL>(D, a, b, smem, red);
    } else if constexpr (KIND == K_NRM) {
        nrm_tile(D, D.ntiles[K_RES], red, true);
    } else if constexpr (KIND == K_CHK) {
        chk_tile(D, io, b, red);
    } else if constexpr (KIND == K_CHKF) {
        nrm_tile(D, D.ntiles[K_CHK], red, false);
    }
}

// The launches of one pass and of the persistent queue (batch_pass.hpp,
// batch_persistent.hpp), per precision.
struct PassLaunch {
    int kind;
    // variant of this launch. Forward x kinds: 1 staged rows, 0 direct loads; y
    // kinds: chunk rows; interface kinds: register rows per lane (the most a
    // problem needs). One kernel for every chunk size takes the registers of 16
    // rows (200, with spills) for all: 158 + 138 us for the y passes of 16
    // problems, 27 million cells, at 8 rows, against 97 + 108 with kernels of
    // their own.
    int sel;
    int refine;  // refinement tile: skipped when the problem converged
    int nblk;
    size_t lds;
    int* d_start;
};

struct PersistArgs {
    const ProblemDesc* desc;
    const ProblemIO* io;
    const int4* tasks;
    const int* kinds;  // kind of each level
    int* counters;     // [nprob][nlevels] completed tiles
    int* ticket;
    int* error;
    int ntasks;
    int nlevels;
    int chunk;  // tasks per ticket
};

void launch_pass64(const PassLaunch& L, const ProblemDesc* desc, const ProblemIO* io, int n, hipStream_t s);
void launch_pass32(const PassLaunch& L, const ProblemDesc* desc, const ProblemIO* io, int n, hipStream_t s);
// the persistent launch over the queue A on a grid that fills the device
void launch_queue64(const PersistArgs& A, size_t lds, int device, hipStream_t s);
void launch_queue32(const PersistArgs& A, size_t lds, int device, hipStream_t s);

}  // namespace psv

// y and z passes of the eigenexpansion solve (Sec. 3.3.1) as block-level
// tile functions (256 threads), shared by the per-pass kernels and the
// persistent batch kernel.
//
// The spectrum keeps one layout, [k][m][n] (plane k, x wavenumber m, y
// wavenumber n; y lines contiguous), through every pass. For every
// wavenumber pair (m, n) != (0, 0) the wall-normal system
//     a_k x_{k-1} + (b_k + lx[m] + ly[n]) x_k + c_k x_{k+1} = R_k
// is solved by a partition method whose chunks are the y tiles themselves:
//  * forward y tile: kc consecutive planes of one m, all n: the FFT along y
//    of its kc lines, then, per n, the local elimination of the chunk's rows
//    (forward sweep, and a backward sweep that reduces row 0), leaving
//      row 0:      A x_{last of previous chunk} + x_first + C x_last = d_0
//      row i:      aa_i x_first + x_i + cc_i x_{i+1} = d_i   (0 < i < kc-1)
//      row kc-1:   aa x_first + x_last + cc x_{first of next chunk} = d_{kc-1}
//    written back in place;
//  * interface pass: per pair, the 2 nc rows (first, last) of its nc chunks
//    form a tridiagonal system with unit diagonal, solved with the Thomas
//    factors precomputed per plan (they do not depend on the data), its two
//    sweeps as affine scans over up to 8 lanes per pair; its tile 0 solves
//    the singular (0, 0) pair in FP64: projection of the right-hand side
//    (removal of its volume-weighted mean), flux integration from the bottom
//    wall, gauge sum_k h_k x_k = 0;
//  * inverse y tile: back substitution of the interior rows from x_first and
//    x_last, then the inverse FFT along y, in place.
// The elimination coefficients of every row are recomputed where they are
// needed (one division per row), so the z solve adds no pass over the
// spectrum: only the interface rows are read and written once more.
#pragma once

#include <type_traits>

#include "internal.hpp"

namespace psv {

// y-line lengths with a compile-time FFT; other lengths (486, 576, 648, 864, 972 and
// those below 16) use the runtime FFT, which ping-pongs between two buffers and
// takes 1.5 to 3 times as long (512x384x96: 190 us per pass against 50). The batched
// kernels hold the first list only.
#define PSV_YZ_SIZES(X) X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(512)
#define PSV_YZ_MORE(X) \
    X(16) X(18) X(24) X(36) X(54) X(72) X(108) X(144) X(162) X(216) X(288) X(324) X(384) X(432) X(768) X(1024)
inline bool yz_batch_compiled(int ny) {
    switch (ny) {
#define PSV_CASE(n) case n:
        PSV_YZ_SIZES(PSV_CASE)
#undef PSV_CASE
        return true;
        default: return false;
    }
}
// Rounding of the FP32 twiddle products, as x_sep; dir: -1 forward, +1 inverse.
template <typename T>
__host__ __device__ constexpr int yz_sep(int ny, int dir) {
    if (sizeof(T) == 8) return 0;
    if (ny == 512) return dir < 0 ? 2 : 0;
#define PSV_CASE(n) if (ny == n) return 0;
    PSV_YZ_SIZES(PSV_CASE)
#undef PSV_CASE
    return 1;
}
inline bool yz_compiled(int ny) {
    switch (ny) {
#define PSV_CASE(n) case n:
        PSV_YZ_MORE(PSV_CASE)
#undef PSV_CASE
        return true;
        default: return yz_batch_compiled(ny);
    }
}

// LDS elements from one line to the next in a compile-time tile (Pad8 layout)
__host__ __device__ constexpr int yz_line_span(int n) { return n + (n + 7) / 8; }
// Threads of a compile-time y tile: 8 elements each up to 2048; larger tiles, of
// which one or two fit a CU, take 512 threads (ny = 384, kc 8: 62 + 55 us at
// 512x384x96 against 72 + 75 with 256), except at kc 16, where the sweeps'
// registers would leave one block per CU (256x256x512 inverse: 151 us against
// 92 with 256).
__host__ __device__ constexpr int yz_threads(int n, int kc) { return n * kc > 2048 && kc <= 8 ? 512 : 256; }

// LDS of a y tile: kc lines (two plain buffers of them for a runtime length)
// and the twiddles
inline size_t yz_lds(int ny, int kc, size_t csz, bool ct) {
    const size_t lines = ct ? (size_t)kc * yz_line_span(ny) : (size_t)2 * kc * ny;
    return (lines + ny) * csz;
}

struct ZArgs {
    int nz, mx, ny;
    FastDiv by_mx, by_ny;  // division by mx and ny
    int kc;          // rows per chunk = planes per y tile (4, 8 or 16)
    int nc;          // chunks per column, ceil(nz / kc)
    double nxny_lz;  // nx * ny * lz
    double lz;
    const double* za;
    const double* zb;
    const double* zc;
    const double* lamx;
    const double* lamy;
    const double* h;
    const double* g;  // centre gaps, g[k] between cells k-1 and k
    double* rhs_mean;
    const void* tab;  // interface factors (layout: ifc_tab_index), in the spectrum's precision
};

// Row k of the system with eigenvalue sum lam; rows k >= nz pad the last
// chunk as identity rows.
struct ZRow {
    double a, b, c;
};
__device__ __forceinline__ ZRow zrow(const ZArgs& z, int k, double lam) {
    // through the constant address space: in a tile k is uniform, and the rows'
    // coefficients then stay in scalar registers whatever else the kernel does
    using K = const __attribute__((address_space(4))) double*;
    if (k < z.nz) return ZRow{((K)z.za)[k], ((K)z.zb)[k] + lam, ((K)z.zc)[k]};
    return ZRow{0.0, 1.0, 0.0};
}

// Rows k0 + i of the system.
__device__ __forceinline__ auto zrows(const ZArgs& z, int k0, double lam) {
    return [&z, k0, lam](int i) { return zrow(z, k0 + i, lam); };
}

// Forward elimination of chunk row i given the reduced row i-1: row i
// becomes aa x_first + x_i + cc x_{i+1} = d (for i = 0, aa couples to the
// previous chunk's last unknown). Returns the pivot reciprocal.
template <typename T>
__device__ __forceinline__ double chunk_fwd(int i, const ZRow& w, T aa_prev, T cc_prev, T& aa,
                                            T& cc) {
    double r;
    if (i < 2) {
        r = rcp_nr(w.b);
        aa = (T)(w.a * r);
    } else {
        r = rcp_nr(w.b - w.a * (double)cc_prev);
        aa = (T)(-w.a * (double)aa_prev * r);
    }
    cc = (T)(w.c * r);
    return r;
}

template <typename T>
__device__ __forceinline__ c2<T> chunk_fwd_rhs(int i, const ZRow& w, double r, c2<T> d, c2<T> dp) {
    if (i < 2) return c2<T>{(T)(d.x * r), (T)(d.y * r)};
    return c2<T>{(T)((d.x - w.a * dp.x) * r), (T)((d.y - w.a * dp.y) * r)};
}

// One backward step over interior row i: with row i+1 in the form
// ab x_first + x_{i+1} + cb x_last = db, row i takes the same form.
template <typename T>
__device__ __forceinline__ void chunk_bwd(T aa, T cc, T& ab, T& cb) {
    ab = aa - cc * ab;
    cb = -cc * cb;
}
template <typename T>
__device__ __forceinline__ c2<T> chunk_bwd_rhs(c2<T> d, T cc, c2<T> db) {
    return c2<T>{d.x - cc * db.x, d.y - cc * db.y};
}
template <typename T>
__device__ __forceinline__ T chunk_row0_pivot(T cc0, T ab1) {
    return (T)1 / ((T)1 - cc0 * ab1);
}

// Local elimination of one system's chunk in registers: forward sweep, and the
// backward sweep that reduces row 0; rows 1..KC-1 keep their forward-swept
// right-hand sides. row(i) gives the system's row i of the chunk.
template <typename T, int KC, typename Row>
__device__ __forceinline__ void chunk_eliminate(Row rows, c2<T>* d) {
    using C = c2<T>;
    T aa[KC], cc[KC];
    C dp{(T)0, (T)0};
    T ap = (T)0, cp = (T)0;
#pragma unroll
    for (int i = 0; i < KC; ++i) {
        const ZRow row = rows(i);
        const double r = chunk_fwd<T>(i, row, ap, cp, aa[i], cc[i]);
        d[i] = chunk_fwd_rhs<T>(i, row, r, d[i], dp);
        dp = d[i];
        ap = aa[i];
        cp = cc[i];
    }
    if constexpr (KC >= 3) {
        C db = d[KC - 2];
        T ab = aa[KC - 2], cb = cc[KC - 2];
#pragma unroll
        for (int i = KC - 3; i >= 1; --i) {
            db = chunk_bwd_rhs<T>(d[i], cc[i], db);
            chunk_bwd<T>(aa[i], cc[i], ab, cb);
        }
        const T r0 = chunk_row0_pivot<T>(cc[0], ab);
        d[0] = C{(d[0].x - cc[0] * db.x) * r0, (d[0].y - cc[0] * db.y) * r0};
    }
}

// Back substitution of one system's chunk in registers: rows 0 and KC-1 hold
// x_first and x_last, rows 1..KC-2 the forward-swept d_i; x_i = d_i - aa_i
// x_first - cc_i x_{i+1}, from i = KC-2 down. Rows i >= nl are padding (x = 0).
template <typename T, int KC, typename Row>
__device__ __forceinline__ void chunk_substitute(Row rows, int nl, c2<T>* d) {
    using C = c2<T>;
    if constexpr (KC >= 3) {
        T aa[KC], cc[KC];
        T ap = (T)0, cp = (T)0;
#pragma unroll
        for (int i = 0; i < KC - 1; ++i) {
            (void)chunk_fwd<T>(i, rows(i), ap, cp, aa[i], cc[i]);
            ap = aa[i];
            cp = cc[i];
        }
        const C xf = d[0];
        C xn = d[KC - 1];
#pragma unroll
        for (int i = KC - 2; i >= 1; --i) {
            xn = i < nl ? C{d[i].x - aa[i] * xf.x - cc[i] * xn.x, d[i].y - aa[i] * xf.y - cc[i] * xn.y}
                        : C{(T)0, (T)0};
            d[i] = xn;
        }
    }
}

// Planes and base of y tile b = c mx + m (chunk c, wavenumber m).
template <typename T>
struct YzTile {
    int m, k0, nl;  // wavenumber, first plane, planes
    size_t SP;      // elements per plane
    c2<T>* base;    // row 0
    __device__ __forceinline__ YzTile(const ZArgs& z, int ny, int kc, c2<T>* spec, int b) {
        const int c = fdiv(b, z.by_mx);
        m = b - c * z.mx;
        k0 = c * kc;
        nl = min(kc, z.nz - k0);
        SP = (size_t)z.mx * ny;
        base = spec + (size_t)k0 * SP + (size_t)m * ny;
    }
};

// Forward y tile b, compile-time ny = N: the FFT along y of the tile's KC
// planes and the local elimination of its N systems. The first stage takes its
// butterflies straight from global memory and the elimination stores its rows
// straight to it (a thread owns system n, so the lanes of a wave store 64
// consecutive elements of a plane): between them the tile passes through LDS
// once per further stage, in place. Against the whole tile staged in LDS first
// and stored from it last: 59 instead of 91 LDS and 393 instead of 553 vector
// instructions per wave (counters); 84.5 -> 82.5 us at 256x256x512 FP64 (541 MB,
// 6.6 TB/s: memory bounds it), 13.4 -> 10.9 at 128^3 (kc 16), where latency does.
template <typename T, int N, int KC, int NT>
__device__ __forceinline__ void yz_fwd_tile_ct(const ZArgs& z, c2<T>* __restrict__ spec,
                                               const c2<T>* __restrict__ tw_g, int b,
                                               unsigned char* smem) {
    using C = c2<T>;
    using P = Pad8;
    constexpr int SEP = yz_sep<T>(N, -1);
    constexpr RadixList RL = radix_list(N);
    constexpr int R = RL.r[0], NB = N / R, TOTAL = KC * NB, IT = (TOTAL + NT - 1) / NT;
    constexpr int TWP = (N + NT - 1) / NT;
    C* buf = reinterpret_cast<C*>(smem);
    constexpr int LS = yz_line_span(N);
    C* tw = buf + KC * LS;  // exp(-2 pi i t / N), t < N
    const YzTile<T> t0(z, N, KC, spec, b);
    {
        C v[IT][R], twr[TWP];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int t = (int)threadIdx.x + it * NT;
            const int line = t / NB, j = t - line * NB;
            if (TOTAL % NT == 0 || t < TOTAL) {
                // within a chunk (at most 16 planes) offsets fit 32 bits
                const unsigned o = (unsigned)(line < t0.nl ? line : 0) * (unsigned)t0.SP + (unsigned)j;
#pragma unroll
                for (int r = 0; r < R; ++r) v[it][r] = at_off(t0.base, o + r * NB);
            }
        }
#pragma unroll
        for (int i = 0; i < TWP; ++i) {
            const int e = (int)threadIdx.x + i * NT;
            twr[i] = tw_g[e < N ? e : 0];
        }
        auto put_tw = [&] {
#pragma unroll
            for (int i = 0; i < TWP; ++i) {
                const int e = (int)threadIdx.x + i * NT;
                if (e < N) tw[e] = twr[i];
            }
        };
        if constexpr (TWP > 1) put_tw();
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int t = (int)threadIdx.x + it * NT;
            const int line = t / NB, j = t - line * NB;
            if (TOTAL % NT == 0 || t < TOTAL) {
                if (line >= t0.nl) {  // planes past the last read as 0
#pragma unroll
                    for (int r = 0; r < R; ++r) v[it][r] = C{(T)0, (T)0};
                }
                bfly_ct<R, -1>(v[it]);
                stockham_store_ct<R, 1, P>(buf + line * LS, j, v[it]);
            }
        }
        if constexpr (TWP == 1) put_tw();
    }
    __syncthreads();
    fft_inplace<N, 1, RL.count, -1, KC, LS, NT, SEP, P>(buf, tw);
    for (int n = threadIdx.x; n < N; n += NT) {
        C d[KC];
        const C* col = buf + P::at(n);
#pragma unroll
        for (int i = 0; i < KC; ++i) d[i] = col[i * LS];
        // the (0,0) pair is solved apart
        if (t0.m != 0 || n != 0) chunk_eliminate<T, KC>(zrows(z, t0.k0, z.lamx[t0.m] + z.lamy[n]), d);
#pragma unroll
        for (int i = 0; i < KC; ++i)
            if (i < t0.nl) at_off(t0.base + (size_t)i * t0.SP, (unsigned)n) = d[i];
    }
}

// Inverse y tile b, compile-time ny = N: x_first and x_last of every system
// sit in rows 0 and KC-1 (written by the interface pass), the interior rows
// hold the forward-swept d_i; back substitution in registers straight from
// global memory, then the inverse FFT along y, whose last stage stores its
// outputs to it.
template <typename T, int N, int KC, int NT>
__device__ __forceinline__ void yz_inv_tile_ct(const ZArgs& z, c2<T>* __restrict__ spec,
                                               const c2<T>* __restrict__ tw_g, int b,
                                               unsigned char* smem) {
    using C = c2<T>;
    using P = Pad8;
    constexpr int SEP = yz_sep<T>(N, 1);
    constexpr RadixList RL = radix_list(N);
    constexpr int LAST = RL.count - 1, R = RL.r[LAST], NB = N / R;
    constexpr int TWP = (N + NT - 1) / NT;
    C* buf = reinterpret_cast<C*>(smem);
    constexpr int LS = yz_line_span(N);
    C* tw = buf + KC * LS;
    const YzTile<T> t0(z, N, KC, spec, b);
    C twr[TWP];
    auto load_tw = [&] {
#pragma unroll
        for (int i = 0; i < TWP; ++i) {
            const int e = (int)threadIdx.x + i * NT;
            twr[i] = tw_g[e < N ? e : 0];
        }
    };
    auto put_tw = [&] {
#pragma unroll
        for (int i = 0; i < TWP; ++i) {
            const int e = (int)threadIdx.x + i * NT;
            if (e < N) tw[e] = twr[i];
        }
    };
    auto rows = [&](int n, C (&d)[KC]) {
#pragma unroll
        for (int i = 0; i < KC; ++i) {
            const C v = at_off(t0.base + (i < t0.nl ? i : 0) * t0.SP, (unsigned)n);
            d[i] = i < t0.nl ? v : C{(T)0, (T)0};
        }
    };
    auto put = [&](int n, C (&d)[KC]) {
        if (t0.m != 0 || n != 0)
            chunk_substitute<T, KC>(zrows(z, t0.k0, z.lamx[t0.m] + z.lamy[n]), t0.nl, d);
        C* col = buf + P::at(n);
#pragma unroll
        for (int i = 0; i < KC; ++i) col[i * LS] = d[i];
    };
    // the twiddles are loaded behind the first system's rows
    if constexpr (TWP > 1) {
        // and stored before the substitution: several of them across its branch go
        // to scratch memory (64x1024x48 step: 99 us, 96 without)
        C first[KC];
        rows((int)threadIdx.x, first);
        load_tw();
        put_tw();
        put((int)threadIdx.x, first);
        for (int n = (int)threadIdx.x + NT; n < N; n += NT) {
            C d[KC];
            rows(n, d);
            put(n, d);
        }
    } else {
        if ((int)threadIdx.x < N) {
            C d[KC];
            rows((int)threadIdx.x, d);
            load_tw();
            put((int)threadIdx.x, d);
        } else {
            twr[0] = C{(T)0, (T)0};
        }
        put_tw();
    }
    __syncthreads();
    fft_inplace<N, 0, LAST, +1, KC, LS, NT, SEP, P>(buf, tw);
    for (int t = threadIdx.x; t < t0.nl * NB; t += NT) {
        const int line = t / NB, j = t - line * NB;
        C v[R];
        stockham_load_ct<R, +1, NB, NB, 1, SEP, P>(buf + line * LS, j, tw, v);
        const unsigned o = (unsigned)line * (unsigned)t0.SP + (unsigned)j;
#pragma unroll
        for (int r = 0; r < R; ++r) at_off(t0.base, o + r * NB) = v[r];
    }
}

// Stages a runtime-length tile's lines (rows past nl read as 0) and the
// twiddles into LDS.
template <typename T, int KC>
__device__ __forceinline__ void yz_load_rt(const ZArgs& z, const YzTile<T>& t0,
                                           const c2<T>* __restrict__ tw_g, c2<T>* buf, c2<T>* tw) {
    using C = c2<T>;
    const int ny = z.ny, nel = KC * ny;
    // one index space: the KC lines, then the ny twiddles; rows past nl
    // load row 0 and are stored as 0
    block_copy<8, C>(
        nel + ny,
        [&](int e) {
            const int i = fdiv(e, z.by_ny), n = e - i * ny;
            return e < nel ? t0.base[(size_t)(i < t0.nl ? i : 0) * t0.SP + n] : tw_g[e - nel];
        },
        [&](int e, C v) {
            if (e < nel)
                buf[e] = fdiv(e, z.by_ny) < t0.nl ? v : C{(T)0, (T)0};
            else
                tw[e - nel] = v;
        });
    __syncthreads();
}

template <typename T>
__device__ __forceinline__ void yz_store_rt(const ZArgs& z, const YzTile<T>& t0, const c2<T>* d) {
    for (int e = threadIdx.x; e < t0.nl * z.ny; e += 256) {
        const int i = fdiv(e, z.by_ny);
        t0.base[(size_t)i * t0.SP + (e - i * z.ny)] = d[e];
    }
}

// The tiles for a runtime ny: lines and FFT in two plain LDS buffers.
template <typename T, int KC>
__device__ __forceinline__ void yz_fwd_tile_rt(const ZArgs& z, const Radices& rad,
                                               c2<T>* __restrict__ spec, const c2<T>* __restrict__ tw_g,
                                               int b, unsigned char* smem) {
    using C = c2<T>;
    const int ny = z.ny;
    C* buf = reinterpret_cast<C*>(smem);
    C* tw = buf + 2 * KC * ny;  // exp(-2 pi i t / ny), t < ny
    const YzTile<T> t0(z, ny, KC, spec, b);
    yz_load_rt<T, KC>(z, t0, tw_g, buf, tw);
    C* r = lds_fft<-1>(buf, buf + KC * ny, ny, KC, ny, rad, tw, ny);
    for (int n = threadIdx.x; n < ny; n += 256) {
        if (t0.m == 0 && n == 0) continue;  // the (0,0) pair is solved apart
        C d[KC];
#pragma unroll
        for (int i = 0; i < KC; ++i) d[i] = r[i * ny + n];
        chunk_eliminate<T, KC>(zrows(z, t0.k0, z.lamx[t0.m] + z.lamy[n]), d);
#pragma unroll
        for (int i = 0; i < KC; ++i) r[i * ny + n] = d[i];
    }
    __syncthreads();
    yz_store_rt(z, t0, r);
}

template <typename T, int KC>
__device__ __forceinline__ void yz_inv_tile_rt(const ZArgs& z, const Radices& rad,
                                               c2<T>* __restrict__ spec, const c2<T>* __restrict__ tw_g,
                                               int b, unsigned char* smem) {
    using C = c2<T>;
    const int ny = z.ny;
    C* buf = reinterpret_cast<C*>(smem);
    C* tw = buf + 2 * KC * ny;
    const YzTile<T> t0(z, ny, KC, spec, b);
    yz_load_rt<T, KC>(z, t0, tw_g, buf, tw);
    for (int n = threadIdx.x; n < ny; n += 256) {
        if (t0.m == 0 && n == 0) continue;
        C d[KC];
#pragma unroll
        for (int i = 0; i < KC; ++i) d[i] = buf[i * ny + n];
        chunk_substitute<T, KC>(zrows(z, t0.k0, z.lamx[t0.m] + z.lamy[n]), t0.nl, d);
#pragma unroll
        for (int i = 1; i < KC - 1; ++i) buf[i * ny + n] = d[i];
    }
    __syncthreads();
    yz_store_rt(z, t0, lds_fft<+1>(buf, buf + KC * ny, ny, t0.nl, ny, rad, tw, ny));
}

// Forward y tile b = c mx + m (chunk c, wavenumber m): FFT along y of planes
// [c KC, c KC + KC) and the local elimination of every system (m, n).
// N = ny as a compile-time constant (NT threads), or 0 for the runtime-length
// FFT (256).
template <typename T, int N, int KC, int NT = 256>
__device__ __forceinline__ void yz_fwd_tile(const ZArgs& z, const Radices& rad,
                                            c2<T>* __restrict__ spec, const c2<T>* __restrict__ tw_g,
                                            int b, unsigned char* smem) {
    if constexpr (N > 0)
        yz_fwd_tile_ct<T, N, KC, NT>(z, spec, tw_g, b, smem);
    else
        yz_fwd_tile_rt<T, KC>(z, rad, spec, tw_g, b, smem);
}

// Inverse y tile b = c mx + m: back substitution of the chunk's rows, then the
// inverse FFT along y.
template <typename T, int N, int KC, int NT = 256>
__device__ __forceinline__ void yz_inv_tile(const ZArgs& z, const Radices& rad,
                                            c2<T>* __restrict__ spec, const c2<T>* __restrict__ tw_g,
                                            int b, unsigned char* smem) {
    if constexpr (N > 0)
        yz_inv_tile_ct<T, N, KC, NT>(z, spec, tw_g, b, smem);
    else
        yz_inv_tile_rt<T, KC>(z, rad, spec, tw_g, b, smem);
}

// Calls f with the compile-time chunk rows matching kc (4, 8 or 16).
template <typename F>
__device__ __forceinline__ void with_kc(int kc, F&& f) {
    if (kc == 4)
        f(std::integral_constant<int, 4>{});
    else if (kc == 8)
        f(std::integral_constant<int, 8>{});
    else
        f(std::integral_constant<int, 16>{});
}

__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// exclusive prefix sum over the 64 lanes
__device__ __forceinline__ double wave_excl_scan(double v) {
    const int lane = threadIdx.x & 63;
    double inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const double t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    return inc - v;
}

// (0,0) column (entry k at col[k * stride]), FP64, as a tile of its own: the
// block (any multiple of 64 threads) stages the real parts, h and g in LDS
// (one global round trip), then one wave solves from there; lane l owns rows [l C, (l+1) C). With
// r~_k = r_k - mean (mean = sum_k h_k r_k / lz, the projection), the flux
// through face k is phi_{k-1} = sum_{j<k} h_j r~_j and
// x_k = sum_{j<=k} g_j phi_{j-1} (x_0 = 0); then the gauge removes
// sum_k h_k x_k / lz.
inline size_t zero_mode_lds(int nz) { return ((size_t)3 * nz + 1) * sizeof(double); }

// Stages the column (all threads; the caller synchronises).
template <typename TS>
__device__ __forceinline__ void zero_mode_stage(const ZArgs& z, const c2<TS>* col, size_t stride,
                                                double* smem) {
    double* r = smem;
    double* hh = r + z.nz;
    double* gg = hh + z.nz;  // [nz + 1]
    for (int k = threadIdx.x; k < z.nz; k += blockDim.x) {
        r[k] = (double)col[(size_t)k * stride].x;
        hh[k] = z.h[k];
    }
    for (int k = threadIdx.x; k <= z.nz; k += blockDim.x) gg[k] = z.g[k];
}

// Solves from the staged values (one wave); put(k, x) stores x_k.
template <typename Put>
__device__ __forceinline__ void zero_mode_solve(const ZArgs& z, const double* smem, Put put) {
    const double* r = smem;
    const double* hh = r + z.nz;
    const double* gg = hh + z.nz;
    const int lane = threadIdx.x & 63;
    const int C = (z.nz + 63) / 64;
    const int k0 = min(lane * C, z.nz), k1 = min(k0 + C, z.nz);
    double s = 0.0;
    for (int k = k0; k < k1; ++k) s += hh[k] * r[k];
    s = wave_sum(s);
    const double mean = s / z.lz;
    if (lane == 0) *z.rhs_mean = s / z.nxny_lz;
    double t = 0.0;
    for (int k = k0; k < k1; ++k) t += hh[k] * (r[k] - mean);
    const double phi0 = wave_excl_scan(t);
    double u = 0.0, phi = phi0;
    for (int k = k0; k < k1; ++k) {
        if (k > 0) u += gg[k] * phi;
        phi += hh[k] * (r[k] - mean);
    }
    const double x0 = wave_excl_scan(u);
    double hx = 0.0, x = x0;
    phi = phi0;
    for (int k = k0; k < k1; ++k) {
        if (k > 0) x += gg[k] * phi;
        phi += hh[k] * (r[k] - mean);
        hx += hh[k] * x;
    }
    const double shift = wave_sum(hx) / z.lz;
    x = x0;
    phi = phi0;
    for (int k = k0; k < k1; ++k) {
        if (k > 0) x += gg[k] * phi;
        phi += hh[k] * (r[k] - mean);
        put(k, x - shift);
    }
}

template <typename TS>
__device__ __forceinline__ void zero_mode_tile(const ZArgs& z, c2<TS>* col, size_t stride,
                                               unsigned char* smem) {
    using T = decltype(c2<TS>::x);
    double* sm = reinterpret_cast<double*>(smem);
    zero_mode_stage<TS>(z, col, stride, sm);
    __syncthreads();
    if (threadIdx.x >= 64) return;
    zero_mode_solve(z, sm, [&](int k, double x) { col[(size_t)k * stride] = c2<TS>{(T)x, (T)0}; });
}

// plane of interface row r: first (even r) or last (odd r) row of chunk r/2
__device__ __forceinline__ int ifc_plane(const ZArgs& z, int r) {
    return (r >> 1) * z.kc + ((r & 1) ? z.kc - 1 : 0);
}

constexpr int IFC_THREADS = 256;  // threads per interface tile

// Lanes per interface system: up to 8 (so that a wave's access to one row
// covers 8 consecutive pairs, whole 128-byte lines of FP64 spectrum), as few
// as leave at most two rows per lane; more than 8 only to keep the rows per
// lane <= 16 (R > 128, i.e. nz / kc > 64).
__host__ __device__ inline int ifc_lanes(int R) {
    int L = 1;
    while (L < 8 && 2 * L < R) L *= 2;
    while (L < 64 && 16 * L < R) L *= 2;
    return L;
}

// Interface systems of one wavenumber pair: R = 2 nc rows on L lanes of a
// wave, Q consecutive rows per lane, spw = 64 / L systems per wave; W waves
// cover the S = mx ny pairs.
struct IfcShape {
    int R, L, Q, spw, W;
};
__host__ __device__ inline IfcShape ifc_shape(int nc, int S) {
    IfcShape h;
    h.R = 2 * nc;
    h.L = ifc_lanes(h.R);
    h.Q = (h.R + h.L - 1) / h.L;
    h.spw = 64 / h.L;
    h.W = (S + h.spw - 1) / h.spw;
    return h;
}

// Factor table layout, wave-blocked: for the wave of systems [w spw, (w+1)
// spw), row slot j < Q and component c (0: -A_r / den_r, 1: -c'_r (0 on the
// last row), 2: 1 / den_r), 64 consecutive entries, one per lane
// (lane = g spw + s - w spw for row r = g Q + j). Each table load of a wave
// is then one contiguous 64-entry access. Slots of no row (s >= S or
// r >= R) are loaded and discarded.
__host__ __device__ inline size_t ifc_tab_index(const IfcShape& h, int s, int r, int c) {
    const int w = s / h.spw, g = r / h.Q, j = r - g * h.Q;
    return (((size_t)w * h.Q + j) * 3 + c) * 64 + g * h.spw + (s - w * h.spw);
}
__host__ __device__ inline size_t ifc_tab_entries(const IfcShape& h) {
    return (size_t)h.W * h.Q * 3 * 64;
}

// One interface system on L lanes of a wave, Q <= QM consecutive rows per
// lane (rows g Q .. g Q + Q - 1 on the lane of group g). With the plan-time
// Thomas factors both sweeps are first-order affine recurrences,
//   forward   d'_r = -(A_r I_r) d'_{r-1} + I_r D_r,         d'_{-1} = 0,
//   backward  x_r  = -c'_r x_{r+1} + d'_r,                    x_R = 0, c'_{R-1} = 0,
// so each lane composes the maps of its rows, the L lanes of a system combine
// theirs by a log2(L)-step scan over the wave (shuffles), and every lane then
// applies its rows from the value coming in. One load and one store per row.
// Padding slots (j >= Q, r >= R) are identity maps in both directions; lanes
// with no system (not act: the zero mode, or past the last) carry identity maps
// through the shuffles and store nothing. tw is the lane's entry of the factor
// table's slot 0, lt loads one; ld(r, rhs) gives the right-hand side of row r where rhs is
// set, st(r, x) takes its solution.
template <typename T, int QM, typename Lt, typename Ld, typename St>
__device__ __forceinline__ void ifc_solve(const ZArgs& z, const IfcShape& h, int lane, int g, bool act,
                                          const T* tw, Lt lt, Ld ld, St st) {
    using C = c2<T>;
    const int R = h.R, L = h.L, Q = h.Q, spw = h.spw;
    const int r0 = g * Q;
    T al[QM], cm[QM];  // forward -A_r I_r, backward -c'_r (identity 1 on padding)
    C d[QM];           // I_r D_r, then d'_r (0 on padding)
    // Every slot is loaded unconditionally (slots j >= Q read slot 0; ld
    // reads some element for a slot without a right-hand side) and masked
    // afterwards, so that all 4 QM loads of a lane are in flight together;
    // loads under per-row branches would each wait.
#pragma unroll
    for (int j = 0; j < QM; ++j) {
        const int r = r0 + j;
        const bool row = act && j < Q && r < R;
        const bool rhs = row && ifc_plane(z, r) < z.nz;
        const T* tj = tw + (size_t)(j < Q ? j : 0) * 3 * 64;
        const T A = lt(tj), Cc = lt(tj + 64), I = lt(tj + 128);
        const C D = ld(r, rhs);
        al[j] = row ? A : (T)1;
        cm[j] = row ? Cc : (T)1;
        d[j] = rhs ? C{I * D.x, I * D.y} : C{(T)0, (T)0};
    }
    // forward: this lane's map d'_{r0-1} -> d'_{r0+Q-1}, then an inclusive scan
    T fa = (T)1;
    C fb{(T)0, (T)0};
#pragma unroll
    for (int j = 0; j < QM; ++j) {
        fa = al[j] * fa;
        fb = C{al[j] * fb.x + d[j].x, al[j] * fb.y + d[j].y};
    }
    for (int off = 1; off < L; off *= 2) {
        const int src = (lane - off * spw) & 63;
        const T pa = __shfl(fa, src, 64);
        const T px = __shfl(fb.x, src, 64), py = __shfl(fb.y, src, 64);
        if (g >= off) {
            fb = C{fa * px + fb.x, fa * py + fb.y};
            fa = fa * pa;
        }
    }
    // d'_{r0-1} is the scanned value of the previous group (0 for g = 0)
    const int prev = (lane - spw) & 63, next = (lane + spw) & 63;
    C v{__shfl(fb.x, prev, 64), __shfl(fb.y, prev, 64)};
    if (g == 0) v = C{(T)0, (T)0};
#pragma unroll
    for (int j = 0; j < QM; ++j) {
        v = C{al[j] * v.x + d[j].x, al[j] * v.y + d[j].y};
        if (act && j < Q && r0 + j < R) d[j] = v;
    }
    // backward: this lane's map x_{r0+Q} -> x_{r0}, then a suffix scan
    T ba = (T)1;
    C bb{(T)0, (T)0};
#pragma unroll
    for (int j = QM - 1; j >= 0; --j) {
        ba = cm[j] * ba;
        bb = C{cm[j] * bb.x + d[j].x, cm[j] * bb.y + d[j].y};
    }
    for (int off = 1; off < L; off *= 2) {
        const int src = (lane + off * spw) & 63;
        const T pa = __shfl(ba, src, 64);
        const T px = __shfl(bb.x, src, 64), py = __shfl(bb.y, src, 64);
        if (g + off < L) {
            bb = C{ba * px + bb.x, ba * py + bb.y};
            ba = ba * pa;
        }
    }
    C x{__shfl(bb.x, next, 64), __shfl(bb.y, next, 64)};
    if (g == L - 1) x = C{(T)0, (T)0};
#pragma unroll
    for (int j = QM - 1; j >= 0; --j) {
        x = C{cm[j] * x.x + d[j].x, cm[j] * x.y + d[j].y};
        const int r = r0 + j;
        if (act && j < Q && r < R && ifc_plane(z, r) < z.nz)
            st(r, x);
    }
}


// The interface systems of tile b >= 1 in the spectrum.
template <typename T, int QM>
__device__ __forceinline__ void ifc_scan(const ZArgs& z, c2<T>* __restrict__ spec, int b) {
    using C = c2<T>;
    const int S = z.mx * z.ny;
    const IfcShape h = ifc_shape(z.nc, S);
    const int spw = h.spw;
    const int lane = (int)threadIdx.x & 63;
    const int g = lane / spw;
    // the wave's first system, and its block of the factor table (the last
    // tile's waves past S read the last block and discard it)
    const int sw = __builtin_amdgcn_readfirstlane((b - 1) * (IFC_THREADS / h.L) +
                                                  ((int)threadIdx.x >> 6) * spw);
    const int s = sw + (lane - g * spw);
    const bool act = s < S && s != 0;
    const T* tw = reinterpret_cast<const T*>(z.tab) +
                  (size_t)min(sw / spw, h.W - 1) * h.Q * 3 * 64 + lane;
    // 32-bit element offsets (every index here is below nx ny nz < 2^31)
    const unsigned us = (unsigned)s, uS = (unsigned)S, s0 = act ? us : 1u;
    ifc_solve<T, QM>(
        z, h, lane, g, act, tw, [](const T* e) { return ld_stream(e); },
        [&](int r, bool rhs) { return spec[rhs ? (unsigned)ifc_plane(z, r) * uS + us : s0]; },
        [&](int r, C x) { spec[(unsigned)ifc_plane(z, r) * uS + us] = x; });
}

// Register rows per lane for R interface rows: 2, 4, 8 or 16 (nz / kc <= 512).
__host__ __device__ inline int ifc_qmax(int R) {
    const int q = (R + ifc_lanes(R) - 1) / ifc_lanes(R);
    return q <= 2 ? 2 : (q <= 4 ? 4 : (q <= 8 ? 8 : 16));
}

// Interface tile b: tile 0 is the (0,0) column; tile b >= 1 solves the
// interface systems of pairs [(b-1) P, b P), P = IFC_THREADS / L. Needs
// blockDim.x == IFC_THREADS and QM >= ifc_qmax(2 nc) (QM = 0: chosen here).
template <typename T, int QM = 0>
__device__ __forceinline__ void ifc_tile(const ZArgs& z, c2<T>* __restrict__ spec, int b,
                                         unsigned char* smem) {
    if (b == 0) {
        zero_mode_tile<T>(z, spec, (size_t)z.mx * z.ny, smem);
        return;
    }
    if constexpr (QM > 0) {
        ifc_scan<T, QM>(z, spec, b);
    } else {
        const int q = ifc_qmax(2 * z.nc);
        if (q == 2)
            ifc_scan<T, 2>(z, spec, b);
        else if (q == 4)
            ifc_scan<T, 4>(z, spec, b);
        else if (q == 8)
            ifc_scan<T, 8>(z, spec, b);
        else
            ifc_scan<T, 16>(z, spec, b);
    }
}

// Interface factors of pair s (plan time; a thread per pair): the coefficients of
// the first and last row of every chunk, from the same sweeps as the y tiles, then
// the Thomas factors, stored as the maps of the interface scans: -A_r / den_r,
// -c'_r = -C_r / den_r, 1 / den_r with den_r = 1 + A_r (-c'_{r-1}) (den_0 = 1).
//
// Without cancellation. Every row is x_i = al x_left + ga x_right (+ d), al and
// ga >= 0, and what they lack of 1, sg = 1 - al - ga, is carried along instead of
// being formed: it starts as -(a + b + c) / -b, which is next to the eigenvalue
// sum over b (the sums' rounding errors are taken in exactly, so it belongs to
// the rounded b that the tiles use), and every pivot is a sum of positive terms,
//     1 - ga' al = (al + sg) + ga (ga' + sg')  for ga' = 1 - al' - sg', and so on.
// As differences the pivots lose the low wavenumbers' sg, whose reciprocal is the
// solve's amplification there: 3.5e-14 of the lowest mode at 128 rows in chunks of
// 8 and 2.2e-14 of 16, 2e-13 to 3e-13 at 1024 rows; summed, 1e-15 to 2e-15 (against
// extended precision). Computed in FP64 whatever the spectrum's precision: an FP32
// recurrence would spoil the corrections of the mixed refinement (256x256x512
// tanh grid: relres 1.8e-10 after one sweep, against 1.1e-11 with the FP64
// table).
template <typename T, int KC>
__device__ __forceinline__ void ifc_table_pair(const ZArgs& z, int s, T* tab) {
    const int S = z.mx * z.ny;
    const IfcShape h = ifc_shape(z.nc, S);
    const int m = s / z.ny, n = s - m * z.ny;
    const double lam = z.lamx[m] + z.lamy[n];
    struct Row {
        double al, ga, sg;
    };
    double t = 0.0;  // 1 + c'_{r-1}
    for (int c = 0; c < z.nc; ++c) {
        ZRow w[KC];
#pragma unroll
        for (int i = 0; i < KC; ++i) w[i] = zrow(z, c * KC + i, 0.0);  // lam is added below
        Row q[KC];
#pragma unroll
        for (int i = 0; i < KC; ++i) {
            const double a = w[i].a, b0 = w[i].b, cc = w[i].c;
            // a + cc = u + eu, b0 + lam = b + eb, exactly
            const double u = a + cc, ua = u - a, eu = (a - (u - ua)) + (cc - ua);
            const double b = b0 + lam, bl = b - b0, eb = (b0 - (b - bl)) + (lam - bl);
            double sg = ((eb - eu) - (u + b0)) - lam;  // -(a + b + cc)
            // where lam vanishes in b the rounded rows are singular (a domain 1e-8 thick)
            // and no FP64 solve of theirs is accurate; the factors stay finite
            if (!(sg > 0.0)) sg = -lam;
            if (i < 2) {
                const double r = rcp_nr(-b);
                q[i] = Row{a * r, cc * r, sg * r};
            } else {
                const double r = rcp_nr((cc + sg) + a * (q[i - 1].al + q[i - 1].sg));
                q[i] = Row{a * q[i - 1].al * r, cc * r, (sg + a * q[i - 1].sg) * r};
            }
            if (c * KC + i >= z.nz) q[i] = Row{0.0, 0.0, 1.0};  // identity rows
        }
        const Row last = q[KC - 1];
        Row b = q[KC - 2];
#pragma unroll
        for (int i = KC - 3; i >= 1; --i)
            b = Row{q[i].al + q[i].ga * b.al, q[i].ga * b.ga, q[i].sg + q[i].ga * b.sg};
        const Row f = q[0];
        const double r0 = rcp_nr((f.al + f.sg) + f.ga * (b.ga + b.sg));
        const Row first{f.al * r0, f.ga * b.ga * r0, (f.sg + f.ga * b.sg) * r0};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const Row x = e == 0 ? first : last;
            const int r = 2 * c + e;
            const double inv = r == 0 ? 1.0 : 1.0 / ((x.ga + x.sg) + x.al * t);
            t = (x.sg + x.al * t) * inv;
            tab[ifc_tab_index(h, s, r, 0)] = (T)(x.al * inv);
            tab[ifc_tab_index(h, s, r, 1)] = (T)(r < h.R - 1 ? x.ga * inv : 0.0);
            tab[ifc_tab_index(h, s, r, 2)] = (T)inv;
        }
    }
}

inline ZArgs make_zargs(const Plan& p, double* mean_out) {
    ZArgs z;
    z.nz = p.nz;
    z.mx = p.mx;
    z.ny = p.ny;
    z.by_mx = fast_div(p.mx);
    z.by_ny = fast_div(p.ny);
    z.kc = p.lp.kc;
    z.nc = (p.nz + p.lp.kc - 1) / p.lp.kc;
    z.lz = p.grid.lz;
    z.nxny_lz = (double)p.nx * p.ny * p.grid.lz;
    z.za = p.t.za;
    z.zb = p.t.zb;
    z.zc = p.t.zc;
    z.lamx = p.t.lamx;
    z.lamy = p.t.lamy;
    z.h = p.t.h;
    z.g = p.t.g;
    z.rhs_mean = mean_out;
    z.tab = p.ifc_tab;
    return z;
}

inline int yz_tiles(const Plan& p) { return p.mx * ((p.nz + p.lp.kc - 1) / p.lp.kc); }
inline int ifc_tiles(const Plan& p) {
    const int per = IFC_THREADS / ifc_lanes(2 * ((p.nz + p.lp.kc - 1) / p.lp.kc));
    return 1 + (p.mx * p.ny + per - 1) / per;
}
inline size_t ifc_lds(const Plan& p) { return zero_mode_lds(p.nz); }

}  // namespace psv

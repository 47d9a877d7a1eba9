// The whole wall-normal solve of a small problem in one launch: a block holds
// all planes of one x wavenumber (ny = 1: of four) in LDS and does there what
// the forward y pass, the interface pass and the inverse y pass do through
// memory, with the same arithmetic. What bounds it is latency: of the 9 us of a
// 128 x 256 problem 4 pass until the planes are in LDS, 1 in the elimination,
// 2 in the interface systems, 1.6 in the substitution and the stores. The three
// launches it replaces take 14.
#include "jobs.hpp"
#include "pass_yz.hpp"

namespace psv {
namespace {

// y lengths of the kernel (ny = 1: two-dimensional problems)
#define PSV_ZF_SIZES(X) X(1) X(16) X(24) X(32) X(48) X(64)

constexpr int ZF_THREADS = 512;
constexpr int ZF_ELEMENTS = 16 * ZF_THREADS;  // elements of a block, 16 per thread

// LDS layout: plane k's systems start at zf_row(k).
template <int N, int KC>
__host__ __device__ constexpr int zf_row(int k) {
    return N > 1 ? k * yz_line_span(N) : k * 4 + k / KC * 4;
}
// The block's LDS, in bytes from its start: y twiddles, the planes, the zero
// mode's column with h and g, the row coefficients, the interface factors.
struct ZfLayout {
    int buf, zero, coef, tab, total;
};
template <typename T>
__host__ __device__ inline ZfLayout zf_layout(int nz, int ny, int kc, const IfcShape& h) {
    const int csz = 2 * sizeof(T);
    const int rows = ny > 1 ? nz * yz_line_span(ny) : nz * 4 + (nz / kc + 1) * 4;
    const int sb = ny > 1 ? ny : 4;
    ZfLayout l;
    l.buf = (ny > 1 ? ny : 0) * csz;
    l.zero = (l.buf + rows * csz + 7) & ~7;
    l.coef = l.zero + (3 * nz + 1) * 8;
    l.tab = l.coef + 3 * nz * 8;
    l.total = l.tab + (sb + h.spw - 1) / h.spw * h.Q * 3 * 64 * (int)sizeof(T);
    if (l.total < 128) l.total = 128;  // a job's block sums
    return l;
}

// One FFT stage over all planes in place; total butterflies at most
// ZF_ELEMENTS / R.
template <int N, int S, int END, int DIR, int SEP, typename C>
__device__ __forceinline__ void zf_stages(C* buf, int nz, const C* tw) {
    using P = Pad8;
    constexpr RadixList RL = radix_list(N);
    if constexpr (S < END) {
        constexpr int R = RL.r[S], NS = radix_prefix(RL, S), NB = N / R, LS = yz_line_span(N);
        constexpr int IT = ZF_ELEMENTS / ZF_THREADS / R + (ZF_ELEMENTS / ZF_THREADS % R ? 1 : 0);
        C v[IT][R];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int t = (int)threadIdx.x + it * ZF_THREADS, line = t / NB;
            if (line < nz)
                stockham_load_ct<R, DIR, NS, NB, N / (NS * R), SEP, P>(buf + line * LS, t - line * NB, tw, v[it]);
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int t = (int)threadIdx.x + it * ZF_THREADS, line = t / NB;
            if (line < nz) stockham_store_ct<R, NS, P>(buf + line * LS, t - line * NB, v[it]);
        }
        __syncthreads();
        zf_stages<N, S + 1, END, DIR, SEP>(buf, nz, tw);
    }
}

template <typename T, int N, int KC>
__global__ void __launch_bounds__(ZF_THREADS) k_zf(ZArgs z, c2<T>* __restrict__ spec,
                                                   const c2<T>* __restrict__ tw_g, int tiles,
                                                   const int* done, Job job) {
    using C = c2<T>;
    using P = Pad8;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if (done && *done) return;
    if ((int)blockIdx.x == tiles) {  // the block past the tiles takes the job
        run_job(job, reinterpret_cast<double*>(smem_raw));
        return;
    }
    constexpr int SEP = N > 1 ? yz_sep<T>(N, -1) : 0;
    constexpr int SB = N > 1 ? N : 4;  // systems per plane of the block
    constexpr int NN = N > 1 ? N : 2;  // (for the transform's constants)
    constexpr RadixList RL = radix_list(NN);
    const int nz = z.nz;
    const IfcShape h = ifc_shape(z.nc, z.mx * z.ny);
    const ZfLayout lay = zf_layout<T>(nz, N, KC, h);
    C* tw = reinterpret_cast<C*>(smem_raw);  // exp(-2 pi i t / N)
    C* buf = reinterpret_cast<C*>(smem_raw + lay.buf);
    double* zs = reinterpret_cast<double*>(smem_raw + lay.zero);
    double* co = reinterpret_cast<double*>(smem_raw + lay.coef);
    T* tab = reinterpret_cast<T*>(smem_raw + lay.tab);
    auto at = [](int n) { return N > 1 ? P::at(n) : n; };
    const int m0 = N > 1 ? (int)blockIdx.x : (int)blockIdx.x * 4;
    const int nsys = N > 1 ? N : min(4, z.mx - m0);
    const unsigned SP = (unsigned)(z.mx * z.ny);
    C* base = spec + m0 * z.ny;
    // Everything the block reads is loaded before anything is written to LDS, so
    // that it waits for memory once: the planes (through the first FFT stage),
    // the row coefficients, the factors of its interface systems (as the table
    // holds them, 64 lanes per row slot and component), h and g. The loops run
    // on only where a thread has more than its first share.
    constexpr int R = RL.r[0], NB = NN / R;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto load_planes = [&](int i, C (&v)[R]) {  // butterfly i
        const int line = i / NB, j = i - line * NB;
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = at_off(base, (unsigned)line * SP + (unsigned)(j + r * NB));
    };
    auto put_planes = [&](int i, C (&v)[R]) {
        bfly_ct<R, -1>(v);
        stockham_store_ct<R, 1, P>(buf + zf_row<N, KC>(i / NB), i % NB, v);
    };
    // ny = 1: element i (past the end the last one). The first four of a thread are
    // variables, as an array of them went to scratch memory, whose store waits for
    // the loads (256 x 512 solve: 21.9 us against 20.3, the 128 x 256 bubble 469 and 428)
    auto load_one = [&](int i) {
        const int e = min(i, nz * 4 - 1), k = e >> 2, n = e & 3;
        return at_off(base, (unsigned)k * SP + (unsigned)(n < nsys ? n : 0));
    };
    auto put_one = [&](int i, C x) {
        if (i < nz * 4) buf[zf_row<N, KC>(i >> 2) + (i & 3)] = x;
    };
    constexpr int PRE = 4;  // elements loaded ahead (ny = 1)
    C v0[R], e0, e1, e2, e3;
    const int tasks = N > 1 ? nz * NB : nz * 4;
    constexpr int STEP = N > 1 ? ZF_THREADS : PRE * ZF_THREADS;
    if constexpr (N > 1) {
        if (tid < tasks) load_planes(tid, v0);
    } else {
        e0 = load_one(tid);
        e1 = load_one(tid + ZF_THREADS);
        e2 = load_one(tid + 2 * ZF_THREADS);
        e3 = load_one(tid + 3 * ZF_THREADS);
    }
    C twr{(T)0, (T)0};
    if (N > 1 && tid < N) twr = tw_g[tid];
    const int kc0 = tid < nz ? tid : 0;
    const double a0 = z.za[kc0], b0 = z.zb[kc0], c0 = z.zc[kc0];
    double h0 = 0.0, g0 = 0.0;
    if (m0 == 0) {
        h0 = z.h[kc0];
        g0 = z.g[tid <= nz ? tid : 0];
    }
    const int g = lane / h.spw;
    const int nw = (SB + h.spw - 1) / h.spw;  // waves of interface systems
    const int ntab = nw * h.Q * 3;
    auto factor = [&](int e) {
        const int w = e / (h.Q * 3), jc = e - w * h.Q * 3;
        const int n = w * h.spw + (lane - g * h.spw), s = N > 1 ? m0 * N + n : m0 + n;
        const int sg = n < nsys ? s : 0, wi = sg / h.spw;
        return reinterpret_cast<const T*>(z.tab)[((size_t)wi * h.Q * 3 + jc) * 64 + g * h.spw +
                                                 (sg - wi * h.spw)];
    };
    constexpr int NWV = ZF_THREADS / 64, TPRE = 6;
    T f0[TPRE];
#pragma unroll
    for (int u = 0; u < TPRE; ++u) f0[u] = factor(min(wave + u * NWV, ntab - 1));
    if constexpr (N > 1) {
        if (tid < tasks) put_planes(tid, v0);
    } else {
        put_one(tid, e0);
        put_one(tid + ZF_THREADS, e1);
        put_one(tid + 2 * ZF_THREADS, e2);
        put_one(tid + 3 * ZF_THREADS, e3);
    }
    if (N > 1 && tid < N) tw[tid] = twr;
    if (tid < nz) {
        co[tid] = a0;
        co[nz + tid] = b0;
        co[2 * nz + tid] = c0;
    }
    if (m0 == 0) {
        if (tid < nz) zs[nz + tid] = h0;
        if (tid <= nz) zs[2 * nz + tid] = g0;
    }
#pragma unroll
    for (int u = 0; u < TPRE; ++u)
        if (wave + u * NWV < ntab) tab[(wave + u * NWV) * 64 + lane] = f0[u];
    for (int i = tid + STEP; i < tasks; i += ZF_THREADS) {
        if constexpr (N > 1) {
            C v[R];
            load_planes(i, v);
            put_planes(i, v);
        } else {
            put_one(i, load_one(i));
        }
    }
    for (int k = tid + ZF_THREADS; k < nz; k += ZF_THREADS) {
        co[k] = z.za[k];
        co[nz + k] = z.zb[k];
        co[2 * nz + k] = z.zc[k];
    }
    if (m0 == 0) {
        for (int k = tid + ZF_THREADS; k < nz; k += ZF_THREADS) zs[nz + k] = z.h[k];
        for (int k = tid + ZF_THREADS; k <= nz; k += ZF_THREADS) zs[2 * nz + k] = z.g[k];
    }
#pragma unroll 4
    for (int e = wave + TPRE * NWV; e < ntab; e += NWV) tab[e * 64 + lane] = factor(e);
    __syncthreads();
    if constexpr (N > 1) zf_stages<N, 1, RL.count, -1, SEP>(buf, nz, tw);
    // a thread's chunk of one system: rows [k0, k0 + nl) of column n
    auto chunks = [&](auto f) {
        for (int t = threadIdx.x; t < z.nc * SB; t += ZF_THREADS) {
            const int c = t / SB, n = t - c * SB, k0 = c * KC, nl = min(KC, nz - k0);
            if (n >= nsys || (m0 == 0 && n == 0)) continue;  // the (0,0) pair is solved apart
            C* col = buf + zf_row<N, KC>(k0) + at(n);
            constexpr int LS = N > 1 ? yz_line_span(NN) : 4;
            const double lam = N > 1 ? z.lamx[m0] + z.lamy[n] : z.lamx[m0 + n] + z.lamy[0];
            C d[KC];
#pragma unroll
            for (int i = 0; i < KC; ++i) d[i] = i < nl ? col[i * LS] : C{(T)0, (T)0};
            f([&](int i) {
                const int k = k0 + i;
                return k < nz ? ZRow{co[k], co[nz + k] + lam, co[2 * nz + k]} : ZRow{0.0, 1.0, 0.0};
            }, nl, d);
#pragma unroll
            for (int i = 0; i < KC; ++i)
                if (i < nl) col[i * LS] = d[i];
        }
    };
    chunks([&](auto rows, int, C* d) { chunk_eliminate<T, KC>(rows, d); });
    if (m0 == 0)  // the (0,0) column's real parts
        for (int k = threadIdx.x; k < nz; k += ZF_THREADS) zs[k] = (double)buf[zf_row<N, KC>(k)].x;
    __syncthreads();
    // interface systems, a wave per spw of them; the zero mode on the last wave
    {
        for (int w = wave; w < nw; w += ZF_THREADS / 64) {
            const int n = w * h.spw + (lane - g * h.spw);
            const bool act = n < nsys && (m0 != 0 || n != 0);
            const T* te = tab + w * h.Q * 3 * 64 + lane;
            auto lt = [](const T* e) { return *e; };
            auto ld = [&](int r, bool rhs) {
                return rhs ? buf[zf_row<N, KC>(ifc_plane(z, r)) + at(n)] : C{(T)0, (T)0};
            };
            auto st = [&](int r, C x) { buf[zf_row<N, KC>(ifc_plane(z, r)) + at(n)] = x; };
            const int q = ifc_qmax(h.R);
            if (q == 2)
                ifc_solve<T, 2>(z, h, lane, g, act, te, lt, ld, st);
            else if (q == 4)
                ifc_solve<T, 4>(z, h, lane, g, act, te, lt, ld, st);
            else if (q == 8)
                ifc_solve<T, 8>(z, h, lane, g, act, te, lt, ld, st);
            else
                ifc_solve<T, 16>(z, h, lane, g, act, te, lt, ld, st);
        }
        if (m0 == 0 && wave == ZF_THREADS / 64 - 1)
            zero_mode_solve(z, zs, [&](int k, double x) { buf[zf_row<N, KC>(k)] = C{(T)x, (T)0}; });
    }
    __syncthreads();
    chunks([&](auto rows, int nl, C* d) { chunk_substitute<T, KC>(rows, nl, d); });
    __syncthreads();
    if constexpr (N > 1) {
        constexpr int LAST = RL.count - 1, R = RL.r[LAST], NB = N / R;
        zf_stages<N, 0, LAST, +1, SEP>(buf, nz, tw);
        for (int t = threadIdx.x; t < nz * NB; t += ZF_THREADS) {
            const int line = t / NB, j = t - line * NB;
            C v[R];
            stockham_load_ct<R, +1, NB, NB, 1, SEP, P>(buf + zf_row<N, KC>(line), j, tw, v);
#pragma unroll
            for (int r = 0; r < R; ++r) at_off(base, (unsigned)line * SP + (unsigned)(j + r * NB)) = v[r];
        }
    } else {
        for (int e = threadIdx.x; e < nz * 4; e += ZF_THREADS) {
            const int k = e >> 2, n = e & 3;
            if (n < nsys) at_off(base, (unsigned)k * SP + (unsigned)n) = buf[zf_row<N, KC>(k) + n];
        }
    }
}

template <typename T, int N, int KC>
void zf_launch(const Plan& p, const ZArgs& z, c2<T>* spec, const c2<T>* tw, const Job& job,
               const int* done, hipStream_t s) {
    const size_t lds = (size_t)zf_layout<T>(p.nz, p.ny, KC, ifc_shape(z.nc, p.mx * p.ny)).total;
    allow_lds(k_zf<T, N, KC>, lds);
    const int tiles = N > 1 ? p.mx : (p.mx + 3) / 4;
    hipLaunchKernelGGL((k_zf<T, N, KC>), dim3(tiles + (job.kind != JOB_NONE ? 1 : 0)), dim3(ZF_THREADS),
                       lds, s, z, spec, tw, tiles, done, job);
}

template <typename T, int N>
void zf_kc(const Plan& p, const ZArgs& z, c2<T>* spec, const c2<T>* tw, const Job& job, const int* done,
           hipStream_t s) {
    switch (p.lp.kc) {
        case 4: zf_launch<T, N, 4>(p, z, spec, tw, job, done, s); break;
        case 8: zf_launch<T, N, 8>(p, z, spec, tw, job, done, s); break;
        default: zf_launch<T, N, 16>(p, z, spec, tw, job, done, s); break;
    }
}

template <typename T>
void zf_dispatch(const Plan& p, const ZArgs& z, c2<T>* spec, const c2<T>* tw, const Job& job,
                 const int* done, hipStream_t s) {
    switch (p.ny) {
#define PSV_CASE(n) case n: zf_kc<T, n>(p, z, spec, tw, job, done, s); break;
        PSV_ZF_SIZES(PSV_CASE)
#undef PSV_CASE
        default: fail(PSV_ERR_INVALID_ARG, "no single-launch z solve for this y length");
    }
}

}  // namespace

bool zf_fits(const Plan& p) {
    switch (p.ny) {
#define PSV_CASE(n) case n:
        PSV_ZF_SIZES(PSV_CASE)
#undef PSV_CASE
        break;
        default: return false;
    }
    const IfcShape h = ifc_shape((p.nz + p.lp.kc - 1) / p.lp.kc, p.mx * p.ny);
    const int lds = p.opts.precision == PSV_MIXED ? zf_layout<float>(p.nz, p.ny, p.lp.kc, h).total
                                                  : zf_layout<double>(p.nz, p.ny, p.lp.kc, h).total;
    if (lds > LDS_MAX_BLOCK) return false;
    // 32^3: 17.0 us per step against 19.4 in three launches, 64x64x32 18.4 and 20.5,
    // 256x16x256 33.6 and 41.1; but 48^3 22.5 and 20.9, 32x32x128 21.0 and 20.5, and
    // more blocks than CUs 33.1 and 32.6 (512x16x64). Two-dimensional: 128x1x512
    // 27.4 and 29.7, 512x1x512 32.5 and 33.1; but 256x1x1024 40.6 and 38.3, 1024x1x512
    // 41.8 and 40.9. Refined ones win at every size that fits (1024x1x1024 137 and 146).
    if (p.ny == 1)
        return p.opts.precision == PSV_MIXED || (p.nz <= 512 && p.mx * p.nz <= 1 << 18);
    return p.mx <= 256 && p.ny * p.nz <= (p.ny <= 16 ? 4096 : 2048);
}

void launch_zf(const Plan& p, bool fp32, double* mean_out, const int* done, hipStream_t s, const Job& job) {
    const ZArgs z = make_zargs(p, mean_out);
    TraceScope ts(p, fp32 ? "z_solve_fp32" : "z_solve_fp64", s);
    if (fp32)
        zf_dispatch<float>(p, z, (float2*)p.spec, p.t.twy32, job, done, s);
    else
        zf_dispatch<double>(p, z, (double2*)p.spec, p.t.twy64, job, done, s);
    PSV_HIP(hipGetLastError());
}

}  // namespace psv

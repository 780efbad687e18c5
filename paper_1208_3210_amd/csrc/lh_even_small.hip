// lh_even_small.hip -- the even path on square grids of 16 to 128 points.
//
// There a call is bound by its launches and by the latency of each kernel's chain of
// loads, exchanges and barriers, not by bytes or operations (32^2 x 64 energies: 0.3 MB
// and 0.9 MFLOP in 30 us).  A slice fits in the LDS of one block (16 to 112 KB, 256
// points do not), so the builder with both forward transforms is one kernel and
// both inverse transforms with the output are another: three launches instead of
// five, and the half-transformed slice never leaves the CU.
// Whole calls, one after another: 32^2 x 64 energies x 32 lags FP64 30.4 -> 18.9 us,
// 64^2 x 256 x 100 FP32 32.1 -> 19.7, 128^2 x 128 x 48 FP32 33.1 -> 23.8,
// 128^2 x 1024 x 400 FP32 82.5 -> 57.3, 128^2 x 256 x 100 FP64 53.5 -> 41.6.
#include <algorithm>

#include "lh_device.h"
#include "lh_regfft.h"

namespace lh {

namespace {

// One slice of N x N points: H + 1 = N / 2 + 1 rows and columns.  Every transform
// line is N points of G threads (RegFFT), all lines of a pass at once.
// Row lines are pairs of rows, consecutive lanes along a line; column lines are
// pairs of neighbouring columns (one complex value per row), ordered tile column,
// thread, tile, so that a wave's accesses cover whole tile rows.
template <typename T, int LOGN>
struct Small {
    // elements per thread: a block's chain is shorter with fewer, until there are more
    // threads than help (builder, us: 32^2 FP32 3.7 with 4, 4.2 with 8, 5.0 with 16;
    // 64^2 FP64 5.2 with 4 and 8, 6.9 with 16; 128^2 allows no less than 8)
    static constexpr int LOGE = LOGN <= 5 ? 2 : 3;
    using F = RegFFT<T, LOGN, false, LOGE, true>;
    static constexpr int N = 1 << LOGN, H = N / 2, G = F::G, C = 16 / sizeof(T);
    static constexpr int NTE = (H + 2 * C) / (2 * C);  // tiles of 2 C columns
    static constexpr int LR = H / 2 + 1, LC = NTE * C;  // row and column lines
    static constexpr int NT = ((LR > LC ? LR : LC) * G + 63) / 64 * 64;
    static constexpr int LINES = NT / G;                // (threads past the last line run on idle lines)
    static constexpr int FS = NTE * 2 * C;              // row stride of the half-transformed slice
    static constexpr size_t LDS = (size_t)(LINES * N + N) * sizeof(cx<T>) + (size_t)(H + 2) * FS * sizeof(T);
    static_assert(NT % (C * G) == 0 && LDS <= 163840, "whole column tiles, LDS of one block");
};

// LDS of a block: transform lines, the twiddles, the half-transformed slice
// f[row][column] (rows 0 .. H, one more so that row pairs are whole).
template <typename T, int LOGN>
struct SmallLds {
    cx<T> *line, *tw;
    T *f;
    __device__ __forceinline__ SmallLds(unsigned char *raw)
    {
        using S = Small<T, LOGN>;
        line = reinterpret_cast<cx<T> *>(raw);
        tw = line + S::LINES * S::N;
        f = reinterpret_cast<T *>(tw + S::N);
    }
};

// P1 and P2 of slice blockIdx.x: the spectral function's row pairs, transformed
// and kept in LDS, then the column pairs, transformed and stored.
template <typename T, int LOGN, bool W>
__device__ __forceinline__ void small_fwd(const double *__restrict__ xi, const Geo &g, double emin, double deps,
                                          double gamma, const cx<T> *__restrict__ twx, T *__restrict__ spec,
                                          const T *__restrict__ rho)
{
    using S = Small<T, LOGN>;
    using F = typename S::F;
    constexpr int N = S::N, H = S::H, G = S::G, E = F::E;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const SmallLds<T, LOGN> l(smem_raw);
    const int tid = threadIdx.x;
    const int j = g.jA + blockIdx.x;
    const double ej = emin + (j + 0.5) * deps;
    const T gp = (T)(gamma / kPi), g2 = (T)(gamma * gamma);
    cx<T> v[E];
    {
        const int p = tid / G, gg = tid % G;
        const bool on = p < S::LR;
        const int ka = on ? 2 * p : 0, kb = on ? min(2 * p + 1, H) : 0;
        double xa[E], xb[E];
#pragma unroll
        for (int s = 0; s < E; ++s) {
            xa[s] = *at32(xi, (unsigned)(ka * N + gg + s * G));
            xb[s] = *at32(xi, (unsigned)(kb * N + gg + s * G));
        }
        for (int i = tid; i < N; i += S::NT) l.tw[tw_swz(i)] = twx[i];
#pragma unroll
        for (int s = 0; s < E; ++s) {
            T a = lorentz((T)(ej - xa[s]), gp, g2), b = lorentz((T)(ej - xb[s]), gp, g2);
            if constexpr (W) {
                a *= *at32(rho, (unsigned)(ka * N + gg + s * G));
                b *= *at32(rho, (unsigned)(kb * N + gg + s * G));
            }
            v[s] = mk<T>(a, b);
        }
        __syncthreads();
        F::run(v, l.line + p * N, l.tw, 0, gg, lds_xor_gfast<N, G>(p));
        if (on) {
#pragma unroll
            for (int s = 0; s < E; ++s) {
                const int n = gg + s * G;
                if (n < S::FS) {
                    l.f[2 * p * S::FS + n] = n <= H ? v[s].x : (T)0;
                    l.f[(2 * p + 1) * S::FS + n] = n <= H ? v[s].y : (T)0;
                }
            }
        }
    }
    __syncthreads();
    {
        const int c = tid % S::C, gg = tid / S::C % G, tile = tid / (S::C * G), ln = tile * S::C + c;
        const bool on = tile < S::NTE;
        const cx<T> *col = reinterpret_cast<const cx<T> *>(l.f) + (on ? ln : 0);
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int n = gg + s * G;
            v[s] = col[(n <= H ? n : N - n) * (S::FS / 2)];
        }
        F::run(v, l.line + ln * N, l.tw, 0, gg, lds_xor_interleaved<T, N>(c, S::C));
        if (on) {
            cx<T> *base = reinterpret_cast<cx<T> *>(spec + (size_t)blockIdx.x * g.slice_e) + tile * g.HyS * S::C + c;
            const int nlo = g.sw ? tile * 2 * S::C : 0;  // (exchange symmetry: the rows the window reads)
#pragma unroll
            for (int s = 0; s < E; ++s) {
                const int n = gg + s * G;
                if (n <= H && n >= nlo) base[n * S::C] = v[s];
            }
        }
    }
}

// P4 and P5 of output plane blockIdx.x (MODE 0: the omega's window slots, blended;
// MODE 1: first-zone plane of that slot, for the RPA path).
template <typename T, int LOGN, int MODE>
__device__ __forceinline__ void small_inv(const T *__restrict__ spec, const Geo &g, const cx<T> *__restrict__ twx,
                                          const PlaneSrc *__restrict__ psrc, double scale, int zx, int zy, int ff,
                                          double ffs, const double2 *__restrict__ ffx, const double2 *__restrict__ ffy,
                                          T *__restrict__ out)
{
    using S = Small<T, LOGN>;
    using F = typename S::F;
    constexpr int N = S::N, H = S::H, G = S::G, E = F::E, VEC = 16 / sizeof(T);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const SmallLds<T, LOGN> l(smem_raw);
    const int tid = threadIdx.x, plane = blockIdx.x;
    const PlaneSrc ps = MODE == 0 ? psrc[plane] : PlaneSrc{plane, -1, 1.0, 0.0};
    const int onx = MODE == 0 ? zx * N : N, ony = MODE == 0 ? zy * N : N;
    T *o = out + (size_t)(MODE == 0 ? plane : g.m_lo + plane) * ony * onx;
    const int nv = onx / VEC;
    if (MODE == 0 && ps.a < 0) {  // the plane is zero
        const lh_u4 z = {0u, 0u, 0u, 0u};
        for (int it = tid; it < ony * nv; it += S::NT) {
            const int Y = it / nv, X = (it - Y * nv) * VEC;
            T *p = o + (size_t)Y * onx + X;
            if ((reinterpret_cast<uintptr_t>(out) & 15) == 0) {
                *reinterpret_cast<lh_u4 *>(p) = z;
            } else {
                for (int i = 0; i < VEC; ++i) p[i] = (T)0;
            }
        }
        return;
    }
    cx<T> v[E];
    {
        const int c = tid % S::C, gg = tid / S::C % G, tile = tid / (S::C * G), ln = tile * S::C + c;
        const bool on = tile < S::NTE;
        const size_t oc = (size_t)(on ? tile : 0) * g.HyS * S::C + c;
        const cx<T> *a = reinterpret_cast<const cx<T> *>(spec + (size_t)ps.a * g.slice_e) + oc;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int n = gg + s * G;
            v[s] = a[(n <= H ? n : N - n) * S::C];
        }
        if (ps.b >= 0 || ps.wa != 1.0) {  // an omega between two lags
            const cx<T> *b = reinterpret_cast<const cx<T> *>(spec + (size_t)(ps.b >= 0 ? ps.b : ps.a) * g.slice_e) + oc;
            const T wa = (T)ps.wa, wb = (T)ps.wb;
#pragma unroll
            for (int s = 0; s < E; ++s) {
                const int n = gg + s * G;
                const cx<T> y = b[(n <= H ? n : N - n) * S::C];
                v[s] = mk<T>(wa * v[s].x + wb * y.x, wa * v[s].y + wb * y.y);
            }
        }
        // (column H's partner is padding, which the half window does not write)
        if (2 * ln + 1 > H) {
#pragma unroll
            for (int s = 0; s < E; ++s) v[s].y = (T)0;
        }
        for (int i = tid; i < N; i += S::NT) l.tw[tw_swz(i)] = twx[i];
        __syncthreads();
        F::run(v, l.line + ln * N, l.tw, 0, gg, lds_xor_interleaved<T, N>(c, S::C));
        if (on) {
            cx<T> *col = reinterpret_cast<cx<T> *>(l.f) + ln;
#pragma unroll
            for (int s = 0; s < E; ++s) {
                const int n = gg + s * G;
                if (n <= H) col[n * (S::FS / 2)] = v[s];
            }
        }
    }
    __syncthreads();
    {
        const int p = tid / G, gg = tid % G;
        const bool on = p < S::LR;
        const T *fa = l.f + (on ? 2 * p : 0) * S::FS, *fb = l.f + (on ? min(2 * p + 1, H) : 0) * S::FS;
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int n = gg + s * G, m = n <= H ? n : N - n;
            v[s] = mk<T>(fa[m], fb[m]);
        }
        F::run(v, l.line + p * N, l.tw, 0, gg, lds_xor_gfast<N, G>(p));
        __syncthreads();
        // the rows 0 .. H in natural order over the lines
        if (on) {
            T *r = reinterpret_cast<T *>(l.line) + 2 * p * N;
            const T sc = (T)scale;
#pragma unroll
            for (int s = 0; s < E; ++s) {
                r[gg + s * G] = v[s].x * sc;
                r[N + gg + s * G] = v[s].y * sc;
            }
        }
    }
    __syncthreads();
    const T *rows = reinterpret_cast<const T *>(l.line);
    const int shx = MODE == 0 ? N / 2 : 0, shy = MODE == 0 ? N / 2 : 0;  // (odd zone counts: N zones / 2 = N / 2 mod N)
    const bool vec = (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    for (int it = tid; it < ony * nv; it += S::NT) {
        const int Y = it / nv, X = (it - Y * nv) * VEC;
        const int qy = (Y + shy) & (N - 1), qx = (X + shx) & (N - 1);
        const T *r = rows + (qy <= H ? qy : N - qy) * N + qx;
        Vec16<T> w;
#pragma unroll
        for (int i = 0; i < VEC; ++i) w.v[i] = r[i];
        if (MODE == 0 && ff) {
            const double2 fy = ffy[Y];
#pragma unroll
            for (int i = 0; i < VEC; ++i) w.v[i] = (T)((double)w.v[i] * form_factor_sq(ffx[X + i], fy, ffs));
        }
        T *p = o + (size_t)Y * onx + X;
        if (vec) {
            *reinterpret_cast<lh_u4 *>(p) = __builtin_bit_cast(lh_u4, w);
        } else {
#pragma unroll
            for (int i = 0; i < VEC; ++i) p[i] = w.v[i];
        }
    }
}

template <typename T, int LOGN, bool W>
__global__ void __launch_bounds__((Small<T, LOGN>::NT))
    k_small_fwd(const double *__restrict__ xi, Geo g, double emin, double deps, double gamma,
                const cx<T> *__restrict__ twx, T *__restrict__ spec, const T *__restrict__ rho)
{
    small_fwd<T, LOGN, W>(xi, g, emin, deps, gamma, twx, spec, rho);
}
template <typename T, int LOGN, bool W>
__global__ void __launch_bounds__((Small<T, LOGN>::NT)) k_small_fwd_batch(const EvenInst *__restrict__ in)
{
    const EvenInst &d = in[blockIdx.z];
    const Geo g = d.g;
    if ((int)blockIdx.x >= g.nS) return;
    small_fwd<T, LOGN, W>(d.xi, g, d.emin, d.deps, d.gamma, (const cx<T> *)d.twx, (T *)d.spec, (const T *)d.rho);
}
template <typename T, int LOGN, int MODE>
__global__ void __launch_bounds__((Small<T, LOGN>::NT))
    k_small_inv(const T *__restrict__ spec, Geo g, const cx<T> *__restrict__ twx, const PlaneSrc *__restrict__ psrc,
                double scale, int zx, int zy, int ff, double ffs, const double2 *__restrict__ ffx,
                const double2 *__restrict__ ffy, T *__restrict__ out)
{
    small_inv<T, LOGN, MODE>(spec, g, twx, psrc, scale, zx, zy, ff, ffs, ffx, ffy, out);
}
template <typename T, int LOGN>
__global__ void __launch_bounds__((Small<T, LOGN>::NT)) k_small_inv_batch(const EvenInst *__restrict__ in)
{
    const EvenInst &d = in[blockIdx.z];
    const Geo g = d.g;
    if ((int)blockIdx.x >= d.nomega) return;
    small_inv<T, LOGN, 0>((const T *)d.spec, g, (const cx<T> *)d.twx, d.psrc, d.scale, d.zx, d.zy, d.ff, d.ffs, d.ffx,
                          d.ffy, (T *)d.out);
}

#define LH_SMALL_SWITCH(v, CALL)          \
    switch (v) {                          \
    case 4: CALL(4); break;               \
    case 5: CALL(5); break;               \
    case 6: CALL(6); break;               \
    case 7: CALL(7); break;               \
    default: return hipErrorInvalidValue; \
    }

template <typename T>
hipError_t fwd_t(const Plan &pl, T *spec, int band, hipStream_t st)
{
    const Geo &g = pl.g;
    const size_t nk = (size_t)g.nkx * g.nky;
#define LH_SF(LG)                                                                                                    \
    do {                                                                                                             \
        using S = Small<T, LG>;                                                                                      \
        const auto k = pl.rho ? &k_small_fwd<T, LG, true> : &k_small_fwd<T, LG, false>;                              \
        hipLaunchKernelGGL(k, dim3(g.nS), dim3(S::NT), S::LDS, st, pl.xi + band * nk, g, pl.p.emin, pl.deps,         \
                           pl.p.gamma, (const cx<T> *)pl.twx, spec,                                                  \
                           pl.rho ? (const T *)pl.rho + band * nk : nullptr);                                        \
    } while (0)
    LH_SMALL_SWITCH(g.logNx, LH_SF)
#undef LH_SF
    return hipGetLastError();
}

template <typename T>
hipError_t inv_t(const Plan &pl, const T *spec, T *out, hipStream_t st)
{
    const Geo &g = pl.g;
    const int ff = pl.p.ff_kind != LINDHARD_FF_NONE;
    const bool rpa = pl.p.want_rpa != 0;
#define LH_SI(LG)                                                                                                    \
    do {                                                                                                             \
        using S = Small<T, LG>;                                                                                      \
        const auto k = rpa ? &k_small_inv<T, LG, 1> : &k_small_inv<T, LG, 0>;                                        \
        hipLaunchKernelGGL(k, dim3(rpa ? g.nL : pl.p.nomega), dim3(S::NT), S::LDS, st, spec, g,                      \
                           (const cx<T> *)pl.twx, pl.d_src, pl.scale, pl.zx, pl.zy, ff, pl.ff_s, pl.ffx, pl.ffy,     \
                           rpa ? (T *)pl.im1 : out);                                                             \
    } while (0)
    LH_SMALL_SWITCH(g.logNx, LH_SI)
#undef LH_SI
    return hipGetLastError();
}

template <typename T>
hipError_t group_t(const Plan *const *pls, int n, const EvenInst *d, bool inv, hipStream_t st)
{
    const Geo &g = pls[0]->g;
    int m = 0;  // slices or omegas of the largest instance
    for (int i = 0; i < n; ++i) m = std::max(m, inv ? (int)pls[i]->p.nomega : pls[i]->g.nS);
#define LH_SG(LG)                                                                                                    \
    do {                                                                                                             \
        using S = Small<T, LG>;                                                                                      \
        const auto k = inv ? &k_small_inv_batch<T, LG>                                                               \
                           : pls[0]->rho ? &k_small_fwd_batch<T, LG, true> : &k_small_fwd_batch<T, LG, false>;       \
        hipLaunchKernelGGL(k, dim3(m, 1, n), dim3(S::NT), S::LDS, st, d);                                            \
    } while (0)
    LH_SMALL_SWITCH(g.logNx, LH_SG)
#undef LH_SG
    return hipGetLastError();
}

}  // namespace

hipError_t launch_small_fwd(const Plan &pl, void *spec, int band, hipStream_t st)
{
    return pl.g.fp64 ? fwd_t<double>(pl, (double *)spec, band, st) : fwd_t<float>(pl, (float *)spec, band, st);
}
hipError_t launch_small_inv(const Plan &pl, const void *spec, void *out, hipStream_t st)
{
    return pl.g.fp64 ? inv_t<double>(pl, (const double *)spec, (double *)out, st)
                     : inv_t<float>(pl, (const float *)spec, (float *)out, st);
}
hipError_t launch_small_group(const Plan *const *pls, int n, const EvenInst *d, bool inv, hipStream_t st)
{
    return pls[0]->g.fp64 ? group_t<double>(pls, n, d, inv, st) : group_t<float>(pls, n, d, inv, st);
}

}  // namespace lh

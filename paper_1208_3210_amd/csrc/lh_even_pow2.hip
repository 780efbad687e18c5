// lh_even_pow2.hip -- builder and column passes of the even path on the half-work
// transform (EvenFFT): axes of 1024 to 4096 points (FP64 columns from 2048; se_rows, se_cols).
//
// Both have the butterfly's inputs computed or loaded by the thread that runs it
// (each value once: the mirror images are never evaluated or read) and leave
// through LDS in natural order.  Against the full transforms (RegFFT) at
// 2048^2 x 512 x 256, ms: builder 0.86 -> 0.63, P2 0.90 -> 0.80, P4 0.47 -> 0.46 in
// FP32, 2.00 -> 1.43, 1.76 -> 1.47 and 0.95 -> 0.87 in FP64; at 4096^2, FP32, 4.5 ->
// 2.7, 4.8 -> 3.1 and 2.8 -> 1.8; at 1024^2, FP32, 0.26 -> 0.16, 0.24 -> 0.18 and 0.13 ->
// 0.10.  The builder is bound by the vector units (75 % busy), the columns by HBM.  The
// last row pass on the same transform (mirrored stores from the butterflies) took 1.8 ms
// against 1.0 and is not kept.
#include <algorithm>

#include "lh_device.h"
#include "lh_evenfft.h"

namespace lh {

namespace {

template <typename T, int LOGN>
constexpr int se_lines()
{
    constexpr int R3 = EvenFFT<T, LOGN>::R3;
    return (sizeof(T) == 4 && R3 >= 8 ? 64 : 32) / R3;
}
template <typename T, int LOGN>
constexpr int se_threads()
{
    return se_lines<T, LOGN>() * EvenFFT<T, LOGN>::TL;
}
// LDS values between lines (col: the lines are interleaved lane by lane, so
// their starts are spread over the banks)
template <typename T, int LOGN>
constexpr int se_stride(bool col)
{
    constexpr int U = sizeof(T) == 4 ? 32 : 8, L = se_lines<T, LOGN>(), LINE = EvenFFT<T, LOGN>::LINE;
    constexpr int want = L <= U ? U / L : 1;
    return col ? LINE + ((want - LINE) % U + U) % U : LINE;
}
template <typename T, int LOGN>
constexpr size_t se_lds(bool col)
{
    return (size_t)(se_lines<T, LOGN>() * se_stride<T, LOGN>(col) + EvenFFT<T, LOGN>::T2) * sizeof(cx<T>);
}
// Place of value n <= N / 2 of a line staged in natural order: two slots of
// padding per 16, so that the stride-16 accesses of the length-P transforms'
// threads spread over the banks.
__device__ __forceinline__ int st_pos(int n) { return n + 2 * (n >> 4); }

// Values v[i] = Z[j], j = k + 16 t + jc(i), of a thread of the length-P transforms
// into the staged line: j <= N / 2 at st_pos(j), the others at st_pos(N - j)
// (which half is fixed by i), both a base of the thread's plus a constant.
// Rows k = 0 and 8 hold every frequency twice: of the upper half they store
// j = N / 2 alone.
template <typename T, int LOGN>
__device__ __forceinline__ void st_scatter(const cx<T> *v, cx<T> *line, int k, int t)
{
    using F = EvenFFT<T, LOGN>;
    cx<T> *lo = line + k + 18 * t, *hi = line + 18 * (F::N / 16) - 18 * t - k - 2;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        constexpr int R3 = F::R3;
        const int jc = R3 * (i / R3) + 16 * (i % R3);  // jc / 16
        const bool up = R3 > 1 ? i % R3 >= R3 / 2 : i >= 8;
        if (!up)
            lo[18 * jc] = v[i];
        else if (k & 7)
            hi[-18 * jc] = v[i];
        else if (jc == F::N / 32 && k == 0 && t == 0)
            lo[18 * jc] = v[i];
    }
}

// |index| of value s of first-pass butterfly g (n = g + P s, folded to n <= N / 2)
template <int P>
__device__ __forceinline__ int se_index(int s, int g)
{
    return s < 8 ? g + P * s : (16 - s) * P - g;
}
template <typename T, int LOGN>
__device__ __forceinline__ void se_fill_t2(cx<T> *t2, const cx<T> *__restrict__ tab, int tid)
{
    using F = EvenFFT<T, LOGN>;
    for (int i = tid; i < F::T2; i += se_threads<T, LOGN>()) t2[i] = tab[F::T1 + i];
}

// y (the butterfly's inputs) -> first pass, rows, length-P transforms -> the
// line in natural order at line2 (st_pos).  Contains block barriers, ends with one.
template <typename T, int LOGN>
__device__ __forceinline__ void se_forward(cx<T> *v, cx<T> *line1, cx<T> *line2, const cx<T> *t2,
                                           const cx<T> *__restrict__ t1, int g, bool act, int q2)
{
    using F = EvenFFT<T, LOGN>;
    if (act) {
        rdft<T, 16, false>(v);
        F::split(v, line1, t1, g);
    }
    __syncthreads();
    const int k = q2 >> F::LOGR3, t = q2 & (F::R3 - 1);
    F::fwd(v, line2 + k * F::PS, t2, t);
    __syncthreads();
    st_scatter<T, LOGN>(v, line2, k, t);
    __syncthreads();
}

// P1: each line is one row ky <= nky / 2 at two consecutive energies, A(e_j) +
// i A(e_j + d): one band value serves both, read again for every pair (held in
// registers it would cost the block its partner on the CU: 80 registers a
// thread, see kSeWaves32).  A block's L consecutive rows fill whole 128-byte lines
// of the tiles (one row at four pairs instead: 0.72 against 0.63 ms; in FP64 3.05
// against 1.43), or with fewer than four rows the blocks of a line run on one XCD.
template <typename T, int LOGN, bool W, bool PAST = false>
__device__ __forceinline__ void se1_body(const double *__restrict__ xi, const Geo &g, double emin, double deps,
                                         double gamma, const cx<T> *__restrict__ tab, T *__restrict__ spec,
                                         const T *__restrict__ rho, int acc, int jc)
{
    using F = EvenFFT<T, LOGN>;
    constexpr int L = se_lines<T, LOGN>(), TH = se_threads<T, LOGN>(), LS = se_stride<T, LOGN>(false);
    constexpr int N = F::N;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem_raw), *t2 = lds + L * LS;
    const int tid = threadIdx.x, line = tid / F::TL, q = tid % F::TL;
    const bool act = q <= F::P / 2;
    const int ky0 = xcd_group(blockIdx.x, L < 4 ? 4 / L : 1) * L, ky = min(ky0 + line, g.Hy - 1);
    if (ky0 >= g.Hy) return;  // padding block (block-uniform)
    se_fill_t2<T, LOGN>(t2, tab, tid);
    const T gp = (T)(gamma / kPi), g2 = (T)(gamma * gamma);
    const int jbeg = g.jA + 2 * jc * (int)blockIdx.y, jend = min(g.jB, jbeg + 2 * jc);
    constexpr int VEC = 16 / sizeof(T), Ce = 2 * VEC;
    // tiles stored side by side: their columns a multiple of 16, so that the
    // staged positions advance by a constant
    constexpr int TS = TH / (2 * L) & ~(16 / Ce - 1);
    const int h = tid & 1, r = (tid >> 1) % L, tile0 = (tid >> 1) / L;
    const int row = ky0 + r;
    for (int j = jbeg; j < jend; j += 2) {
        const int qo = q + opaque_zero();
        const double ea = emin + (j + 0.5) * deps, eb = emin + (j + 1.5) * deps;
        cx<T> v[16];
        if (act) {
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const unsigned o = (unsigned)(ky * N + se_index<F::P>(s, qo));
                const double xb = *at32(xi, o);
                v[s] = mk<T>(lorentz((T)(ea - xb), gp, g2), lorentz((T)(eb - xb), gp, g2));
                if constexpr (W) v[s] = cscale(v[s], *at32(rho, o));
            }
        }
        se_forward<T, LOGN>(v, lds + line * LS, lds + line * LS, t2, tab, qo, act, qo);
        // 16-byte pieces (half h of tile row r): a thread keeps its h and r and
        // walks the tiles, TS at a time
        if (tid < TS * 2 * L && row < g.Hy) {
            const bool two = j + 1 < jend;
            T *da = spec + (size_t)(j - g.jA) * g.slice_e;
            unsigned o = (unsigned)((tile0 * g.HyS + row) * g.Ce + h * VEC);
            const cx<T> *zp = lds + r * LS + st_pos(tile0 * Ce + h * VEC);
            for (int tile = tile0; tile < g.NTe; tile += TS, o += TS * g.HyS * Ce, zp += TS * Ce / 16 * 18) {
                Vec16<T> a, b;
                if (tile < g.NTe - 1) {
#pragma unroll
                    for (int i = 0; i < VEC; i += VEC / 2) {
                        const Vec16<T> z = __builtin_bit_cast(Vec16<T>, *reinterpret_cast<const lh_u4 *>(zp + i));
#pragma unroll
                        for (int e = 0; e < VEC / 2; ++e) {
                            a.v[i + e] = z.v[2 * e];
                            b.v[i + e] = z.v[2 * e + 1];
                        }
                    }
                } else {  // the last tile holds n = N / 2 alone
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {
                        const cx<T> z = i + h == 0 ? zp[0] : mk<T>((T)0, (T)0);
                        a.v[i] = z.x;
                        b.v[i] = z.y;
                    }
                }
                lh_u4 *pa = reinterpret_cast<lh_u4 *>(at32(da, o)), *pb = reinterpret_cast<lh_u4 *>(at32(da + g.slice_e, o));
                if (acc) {  // add this band to the earlier ones
                    const Vec16<T> oa = __builtin_bit_cast(Vec16<T>, *pa);
                    const Vec16<T> ob = two ? __builtin_bit_cast(Vec16<T>, *pb) : oa;
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {
                        a.v[i] += oa.v[i];
                        b.v[i] += ob.v[i];
                    }
                }
                store_past<PAST>(pa, __builtin_bit_cast(lh_u4, a));
                if (two) store_past<PAST>(pb, __builtin_bit_cast(lh_u4, b));
            }
        }
        __syncthreads();
    }
}

// Waves per SIMD the FP32 kernels are compiled for: a block of nine waves puts
// three on one SIMD, so two blocks per CU (18 waves) need room for six.
constexpr int kSeWaves32 = 6;

template <typename T, int LOGN, bool W, bool PAST>
__global__ void __launch_bounds__((se_threads<T, LOGN>()), (sizeof(T) == 4 ? kSeWaves32 : 2))
    k_se1(const double *__restrict__ xi, Geo g, double emin, double deps, double gamma, const cx<T> *__restrict__ tab,
          T *__restrict__ spec, const T *__restrict__ rho, int acc, int jc)
{
    se1_body<T, LOGN, W, PAST>(xi, g, emin, deps, gamma, tab, spec, rho, acc, jc);
}
template <typename T, int LOGN, bool W>
__global__ void __launch_bounds__((se_threads<T, LOGN>()), (sizeof(T) == 4 ? kSeWaves32 : 2))
    k_se1_batch(const EvenInst *__restrict__ in, int jc)
{
    const EvenInst &d = in[blockIdx.z];
    const Geo g = d.g;
    if ((int)blockIdx.y * 2 * jc >= g.nS) return;
    se1_body<T, LOGN, W>(d.xi, g, d.emin, d.deps, d.gamma, (const cx<T> *)d.evx, (T *)d.spec, (const T *)d.rho, 0, jc);
}

// P2 (INV false), P4 (INV true): each line is a pair of neighbouring real columns
// of a tile (one complex value per row), the lines of a tile interleaved lane by
// lane so that a wave's loads and stores cover whole tile rows.  In place.  The inverse
// takes the padding columns (rx > nkx/2) as zero (see ecol_body).
template <typename T, int LOGN, bool INV, bool PAST = false>
__device__ __forceinline__ void secol_body(T *__restrict__ spec, const Geo &g, const cx<T> *__restrict__ tab)
{
    using F = EvenFFT<T, LOGN>;
    constexpr int L = se_lines<T, LOGN>(), LS = se_stride<T, LOGN>(true);
    constexpr int C = 16 / sizeof(T), N = F::N;
    static_assert(L % C == 0, "whole tiles");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem_raw), *t2 = lds + L * LS;
    const int tid = threadIdx.x;
    const int line = tid % L, q = tid / L;            // first pass
    const int line2 = tid / F::TL, q2 = tid % F::TL;  // length-P transforms
    const int tile0 = blockIdx.x * (L / C), tile = tile0 + line / C, c = line % C;
    const int rx = tile * g.Ce + 2 * c;  // first column of the pair
    const bool in = tile < g.NTe && (!INV || rx <= g.L), act = q <= F::P / 2 && in;
    se_fill_t2<T, LOGN>(t2, tab, tid);
    cx<T> *base = reinterpret_cast<cx<T> *>(spec + (size_t)blockIdx.y * g.slice_e);
    const unsigned o0 = (unsigned)((act ? tile : 0) * g.HyS * C + c);
    cx<T> v[16];
    if (act) {
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = *at32(base, o0 + se_index<F::P>(i, q) * C);
        // (a branch of the last block only: on every path it takes registers)
        if (INV && tile0 + L / C >= g.NTe) {
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i].y = rx + 1 > g.L ? (T)0 : v[i].y;
        }
    }
    se_forward<T, LOGN>(v, lds + line * LS, lds + line2 * LS, t2, tab, q, act, q2);
    if (q > 8 * F::R3 || !in) return;
    // rows n = q + 8 R3 i (and n = N / 2), the lines side by side; with the
    // exchange symmetry the window reads the rows ry >= Ce tile only
    const int nlo = INV || !g.sw ? 0 : tile * g.Ce, i1 = q < 8 * F::R3 ? 16 : 1;
    const cx<T> *zp = lds + line * LS + st_pos(q < 8 * F::R3 ? q : N / 2);
    const int n0 = q < 8 * F::R3 ? q : N / 2;
    const unsigned oo = (unsigned)(tile * g.HyS * C + c + n0 * C);
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (i < i1 && n0 + 8 * F::R3 * i >= nlo)
            store_past<PAST>(at32(base, oo + 8 * F::R3 * i * C), zp[9 * F::R3 * i]);
}
template <typename T, int LOGN, bool INV, bool PAST>
__global__ void __launch_bounds__((se_threads<T, LOGN>()), (sizeof(T) == 4 ? kSeWaves32 : 2))
    k_secol(T *__restrict__ spec, Geo g, const cx<T> *__restrict__ tab)
{
    secol_body<T, LOGN, INV, PAST>(spec, g, tab);
}
template <typename T, int LOGN, bool INV>
__global__ void __launch_bounds__((se_threads<T, LOGN>()), (sizeof(T) == 4 ? kSeWaves32 : 2))
    k_secol_batch(const EvenInst *__restrict__ in)
{
    const EvenInst &d = in[blockIdx.z];
    const Geo g = d.g;
    if ((int)blockIdx.y >= (INV ? g.nL : g.nS)) return;
    secol_body<T, LOGN, INV>((T *)d.spec, g, (const cx<T> *)d.evy);
}

inline unsigned cdiv(long a, long b) { return (unsigned)((a + b - 1) / b); }

#define LH_SE_SWITCH(v, CALL)             \
    switch (v) {                          \
    case 10: CALL(10); break;             \
    case 11: CALL(11); break;             \
    case 12: CALL(12); break;             \
    default: return hipErrorInvalidValue; \
    }
// columns (FP64 from 2048 points: se_axis_y)
#define LH_SE_COLS(v, CALL)                     \
    if constexpr (sizeof(T) == 4) {             \
        LH_SE_SWITCH(v, CALL)                   \
    } else {                                    \
        switch (v) {                            \
        case 11: CALL(11); break;               \
        case 12: CALL(12); break;               \
        default: return hipErrorInvalidValue;   \
        }                                       \
    }

// Pairs of energies a builder block of rows walks: up to four, whose twiddles and band
// rows (in L2) then serve them all (2048^2 x 512: 0.70 ms at 1, 0.63 at 4, 0.66 at 8), as
// long as 2048 blocks remain (4096 x 256 x 8 slices: 33 us at 4, 17 at 1).  Results do
// not depend on it.
template <typename T, int LOGN>
int se1_jc(long blocks, long pairs)
{
    return LOGN >= 11 ? (int)std::max(1L, std::min(4L, blocks * pairs / 2048)) : 1;
}

// Slices of 1 GB and more in all, four times the last-level cache, are stored past
// the caches: the next pass starts at their beginning, which is evicted by then
// either way, and the pass's own reads stay.  2048^2 x 512 x 256, ms: builder
// 0.64 -> 0.61, P2 0.76 -> 0.71, P4 0.43 -> 0.42, FP64 1.44 -> 1.41, 1.48 -> 1.40 and 0.86 ->
// 0.83; 1024^2 x 1024 FP32 0.27 -> 0.28 and 0.36 -> 0.30, 1024 x 2048 x 600 P2 0.53 -> 0.50.
// A call with 134 MB of slices (2048^2, 16 lags) would go 259 -> 274 us, one with 0.5 GB
// of FP64 ones 973 -> 997.
inline bool se_past(const Geo &g, int slices)
{
    return (size_t)slices * g.slice_e * (g.fp64 ? 8 : 4) >= (size_t)1 << 30;
}

template <typename T>
hipError_t se1_t(const Plan &pl, T *spec, int band, int acc, hipStream_t st)
{
    const Geo &g = pl.g;
    const size_t nk = (size_t)g.nkx * g.nky;
    const int pairs = (g.nS + 1) / 2;
#define LH_SE1(LG)                                                                                                   \
    do {                                                                                                             \
        constexpr int L = se_lines<T, LG>(), GR = L < 4 ? 4 / L : 1;                                                 \
        const unsigned nx = cdiv(cdiv(g.Hy, L), 8 * GR) * 8 * GR;                                                    \
        const int jc = se1_jc<T, LG>(nx, pairs);                                                                     \
        const dim3 grid(nx, cdiv(pairs, jc));                                                                        \
        const bool past = se_past(g, g.nS);                                                                          \
        const auto k = pl.rho ? (past ? &k_se1<T, LG, true, true> : &k_se1<T, LG, true, false>)                      \
                              : (past ? &k_se1<T, LG, false, true> : &k_se1<T, LG, false, false>);                   \
        hipLaunchKernelGGL(k, grid, dim3(se_threads<T, LG>()), (se_lds<T, LG>(false)), st, pl.xi + band * nk, g,     \
                           pl.p.emin, pl.deps, pl.p.gamma, (const cx<T> *)pl.evx, spec,                              \
                           pl.rho ? (const T *)pl.rho + band * nk : nullptr, acc, jc);                               \
    } while (0)
    LH_SE_SWITCH(g.logNx, LH_SE1)
#undef LH_SE1
    return hipGetLastError();
}

template <typename T>
hipError_t secol_t(const Plan &pl, T *spec, int n, bool inv, hipStream_t st)
{
    const Geo &g = pl.g;
#define LH_SEC(LG)                                                                                                   \
    do {                                                                                                             \
        constexpr int TB = se_lines<T, LG>() / (16 / (int)sizeof(T));                                                \
        const dim3 grid(cdiv(g.NTe, TB), n);                                                                         \
        const bool past = se_past(g, n);                                                                             \
        const auto k = inv ? (past ? &k_secol<T, LG, true, true> : &k_secol<T, LG, true, false>)                     \
                           : (past ? &k_secol<T, LG, false, true> : &k_secol<T, LG, false, false>);                  \
        hipLaunchKernelGGL(k, grid, dim3(se_threads<T, LG>()), (se_lds<T, LG>(true)), st, spec, g,                   \
                           (const cx<T> *)pl.evy);                                                            \
    } while (0)
    LH_SE_COLS(g.logNy, LH_SEC)
#undef LH_SEC
    return hipGetLastError();
}

// The same for a batched group (equal grids): grids span the largest instance.
template <typename T>
hipError_t se_group_t(const Plan *const *pls, int n, const EvenInst *d, int pass, hipStream_t st)
{
    const Geo &g = pls[0]->g;
    int m = 0;  // slices or lags of the largest instance
    for (int i = 0; i < n; ++i)
        m = std::max(m, pass == 4 ? pls[i]->g.nL : pls[i]->g.nS);
    if (pass == 1) {
#define LH_SE1(LG)                                                                                                   \
    do {                                                                                                             \
        constexpr int L = se_lines<T, LG>(), GR = L < 4 ? 4 / L : 1;                                                 \
        const unsigned nx = cdiv(cdiv(g.Hy, L), 8 * GR) * 8 * GR;                                                    \
        const int jc = se1_jc<T, LG>(nx, (long)n * ((m + 1) / 2));                                                   \
        const dim3 grid(nx, cdiv((m + 1) / 2, jc), n);                                                               \
        const auto k = pls[0]->rho ? &k_se1_batch<T, LG, true> : &k_se1_batch<T, LG, false>;                         \
        hipLaunchKernelGGL(k, grid, dim3(se_threads<T, LG>()), (se_lds<T, LG>(false)), st, d, jc);                   \
    } while (0)
        LH_SE_SWITCH(g.logNx, LH_SE1)
#undef LH_SE1
    } else {
#define LH_SEC(LG)                                                                                                   \
    do {                                                                                                             \
        constexpr int TB = se_lines<T, LG>() / (16 / (int)sizeof(T));                                                \
        const auto k = pass == 4 ? &k_secol_batch<T, LG, true> : &k_secol_batch<T, LG, false>;                       \
        hipLaunchKernelGGL(k, dim3(cdiv(g.NTe, TB), m, n), dim3(se_threads<T, LG>()), (se_lds<T, LG>(true)), st, d); \
    } while (0)
        LH_SE_COLS(g.logNy, LH_SEC)
#undef LH_SEC
    }
    return hipGetLastError();
}

}  // namespace

// Rows of 1024 and 2048 points take it from 512 blocks on (two per CU), and from 16
// blocks of rows, so that the last one's missing rows cost little: with fewer the full
// transform's smaller blocks are faster (1024^2, us, FP32: 2 slices 8.9 against 10.5,
// 8 slices 14.2 against 15.9, 32 slices 30.6 against 23.3; FP64 11.3 and 14.0, 21.6
// and 22.6, 51.8 and 37.8; 512 slices of 33 rows: 1024 x 64 FP32 28.5 and 30.0, 2048 x 64
// FP64 83 and 92; of 129 rows: 1024 x 256 FP32 70 and 56, 2048 x 256 FP64 267 and 237).
bool se_rows(const Geo &g)
{
    if (!se_axis_x(g)) return false;
    if (g.logNx >= 12) return true;
    const int R3 = 1 << (g.logNx - 8), L = (g.fp64 || R3 < 8 ? 32 : 64) / R3;
    return g.Hy >= 16 * L && (long)cdiv(g.Hy, L) * ((g.nS + 1) / 2) >= 512;
}
// Columns: FP32 always (64 x 1024 x 1 slice 7.7 and 7.9 us, 1024^2 x 64 33 and 29).  In
// FP64 the full transform is faster at 512 and 1024 points (512^2 x 64 24.6 us against
// 27.4, 1024^2 x 256 243 against 256), and at 2048 with less than 128 blocks (256 x
// 2048, 4 slices 10.4 and 11.8 us, 16 slices 18.8 and 17.2, 256 slices 128 and 116).
bool se_cols(const Geo &g, int n)
{
    if (!se_axis_y(g)) return false;
    // (2048 points in FP64: four lines, so two tiles, to a block)
    return !g.fp64 || g.logNy >= 12 || (long)cdiv(g.NTe, 2) * n >= 128;
}

hipError_t launch_se_group(const Plan *const *pls, int n, const EvenInst *d, int pass, hipStream_t st)
{
    return pls[0]->g.fp64 ? se_group_t<double>(pls, n, d, pass, st) : se_group_t<float>(pls, n, d, pass, st);
}

hipError_t launch_se1(const Plan &pl, void *spec, int band, int acc, hipStream_t st)
{
    return pl.g.fp64 ? se1_t<double>(pl, (double *)spec, band, acc, st) : se1_t<float>(pl, (float *)spec, band, acc, st);
}
hipError_t launch_secol(const Plan &pl, void *spec, int n, bool inv, hipStream_t st)
{
    return pl.g.fp64 ? secol_t<double>(pl, (double *)spec, n, inv, st) : secol_t<float>(pl, (float *)spec, n, inv, st);
}
}  // namespace lh

// lh_even_any.hip -- the mirror-symmetric path on grids whose sizes are not
// powers of two.
//
// Every transform maps real even lines to real even lines (lh_kernels.hip, the
// even passes), two of them packed as a + i b.  A line of N points runs as
// Bluestein's chirp convolution over centred indices: with H = floor(N / 2) and
// b_n = exp(i pi n^2 / N),
//   C_k = conj(b_k) sum_{|n| <= H} x_n conj(b_n) b_{k - n},  k = 0 .. H
// (x_{+-H} halved when N is even, the two ends being one point).  Chirp and
// input are even in n, so the convolution of length M = 2^logM >= 4 H is a
// forward transform, a product with an even spectrum and an inverse transform
// of even sequences: EvenFFT, 9/16 of the work of the full transforms, and the
// forward and inverse passes of the grid are the same kernel.  Only the quarter
// plane rx <= nkx / 2, ry <= nky / 2 of real values is stored (the layout of
// the even path), a quarter of the bytes of the complex half plane, and the
// energy window is the even path's.
//
// 2049^2 points x 512 energies x 256 lags with momentum density, FP32, against
// the full complex Bluestein passes (ms): P1 16.7 -> 2.9, P2 11.1 -> 2.3, window
// 7.3 -> 0.6, P4 5.7 -> 1.2, P5 9.7 -> 2.1; a call 50.6 -> 9.1.  300 x 257 x 128 x 64
// in FP64: 0.66 -> 0.19.  Bound by the vector units (59 - 68 % busy) and the
// latency of the exchanges at eighteen waves per CU; 300 x 257 in FP64 by that latency
// alone (vector units 14 - 22 % busy, blocks of 4.5 waves).
#include <algorithm>

#include "lh_device.h"
#include "lh_evenfft.h"

namespace lh {

namespace {

// Tables of one axis: chirp b_n (n <= H), the chirp spectrum / M in the order
// a thread of EvenFFT holds it (value i of thread q at i TL + q), and the
// twiddles T1 then T2 of EvenFFT.
struct EvTab {
    const void *b, *h, *t;
    int n;
};

// Threads of a block: nine waves of FP32 lines (78 KB of LDS: two blocks per
// CU), half of that in FP64 or for the short transforms.  A block of an odd
// number of waves puts three of them on one SIMD, so two blocks per CU need at
// most 80 registers a thread (with 96: one block, P5 2.1 -> 2.7 ms); two lines per
// thread in half the waves measured slower (11.0 -> 13.9 ms a call).
template <typename T, int LOGM>
constexpr int ev_lines()
{
    constexpr int R3 = EvenFFT<T, LOGM>::R3;
    return (sizeof(T) == 4 && R3 >= 8 ? 64 : 32) / R3;
}
template <typename T, int LOGM>
constexpr int ev_threads()
{
    return ev_lines<T, LOGM>() * EvenFFT<T, LOGM>::TL;
}
// Pairs of energies a block of the builder takes side by side: more of them share
// the band values, fewer leave longer pieces of the 128-byte lines to a block
// (2049^2 x 512: 3.07 ms with one, 2.89 with two, 3.56 with four).
constexpr int kEvPairs = 2;
// LDS values between lines: the row passes run consecutive lanes along one
// line; the column passes interleave the lines lane by lane, so there the line
// starts are spread over the banks (32 or 8 consecutive slots are served at once).
template <typename T, int LOGM>
constexpr int ev_stride(bool col)
{
    constexpr int U = sizeof(T) == 4 ? 32 : 8, L = ev_lines<T, LOGM>(), LINE = EvenFFT<T, LOGM>::LINE;
    constexpr int want = L <= U ? U / L : 1;
    return col ? LINE + ((want - LINE) % U + U) % U : LINE;
}
template <typename T, int LOGM>
constexpr size_t ev_lds(bool col)
{
    return (size_t)(ev_lines<T, LOGM>() * ev_stride<T, LOGM>(col) + EvenFFT<T, LOGM>::T2) * sizeof(cx<T>);
}

// The first pass reads x_n for n = g + P s, |n| <= H <= M / 4: s = 0 .. 3 (and 4
// for g = 0) and the mirrored s = 12 .. 15, n = -((16 - s) P - g).
constexpr int kNz = 9;
constexpr unsigned kNzMask = 0xF01Fu;
template <int P>
__device__ __forceinline__ int ev_index(int i, int g)
{
    return i < 5 ? g + P * i : (9 - i) * P - g;
}
__host__ __device__ constexpr int ev_slot(int i) { return i < 5 ? i : i + 7; }

// conj(b_n) times the weight of input n: 0 past H, 1/2 at the end point of an
// even N.
template <typename T>
__device__ __forceinline__ cx<T> ev_chirp(const EvTab &t, int n, bool in)
{
    const cx<T> b = *at32((const cx<T> *)t.b, in ? n : 0);
    const T w = !in ? (T)0 : 2 * n == t.n ? (T)0.5 : (T)1;
    return mk<T>(b.x * w, -b.y * w);
}

// From the chirped inputs of butterfly g (x[i], i < 9) to the outputs C_n at
// the same nine places, through the line's LDS rows.  Contains block barriers;
// the LDS may be reused after the caller's next one.
// TOGETHER: the closing chirp loads without branches, all in flight at once (the
// builder: 4.1 -> 3.6 ms at 2049^2 x 512; in the last row pass the registers they
// take spill: 2.1 -> 2.7 ms).
template <typename T, int LOGM, bool TOGETHER = false>
__device__ __forceinline__ void ev_convolve(cx<T> *x, cx<T> *line1, cx<T> *line2, const cx<T> *t2, const EvTab &tab,
                                            int g, bool act, int q2)
{
    using F = EvenFFT<T, LOGM>;
    const cx<T> *t1 = (const cx<T> *)tab.t, *h = (const cx<T> *)tab.h;
    if (act) {
        cx<T> v[16];
#pragma unroll
        for (int i = 0; i < kNz; ++i) v[ev_slot(i)] = x[i];
        rdft_nz<T, 16, false, kNzMask>(v);
        F::split(v, line1, t1, g);
    }
    __syncthreads();
    {
        cx<T> v[16];
        cx<T> *row = line2 + (q2 >> F::LOGR3) * F::PS;
        const int t = q2 & (F::R3 - 1);
        F::fwd(v, row, t2, t);
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = cmul(v[i], *at32(h, i * F::TL + q2));
        F::inv(v, row, t2, t);
    }
    __syncthreads();
    if (act) {
        // the twiddles and chirps of the first pass are read again, not held in
        // registers through the length-P transforms
        g += opaque_zero();
        cx<T> v[16];
        F::merge(v, line1, t1, g);
        rdft<T, 16, true>(v);
        const int H = tab.n / 2;
#pragma unroll
        for (int i = 0; i < kNz; ++i) {
            const int n = ev_index<F::P>(i, g);
            if constexpr (TOGETHER)
                x[i] = cmul(v[ev_slot(i)], cconj(*at32((const cx<T> *)tab.b, n <= H ? n : 0)));
            else
                x[i] = n <= H ? cmul(v[ev_slot(i)], cconj(*at32((const cx<T> *)tab.b, n))) : mk<T>((T)0, (T)0);
        }
    }
}

// Streamed values: kept out of the L1, which holds the tables.
template <typename T>
__device__ __forceinline__ cx<T> load_nt(const cx<T> *p)
{
    typedef T V2 __attribute__((ext_vector_type(2)));
    const V2 v = __builtin_nontemporal_load(reinterpret_cast<const V2 *>(p));
    return mk<T>(v.x, v.y);
}
template <typename T>
__device__ __forceinline__ void store_nt(cx<T> *p, cx<T> z)
{
    typedef T V2 __attribute__((ext_vector_type(2)));
    __builtin_nontemporal_store(V2{z.x, z.y}, reinterpret_cast<V2 *>(p));
}

// T2 into LDS (the caller's next barrier makes it visible)
template <typename T, int LOGM>
__device__ __forceinline__ void ev_fill_t2(cx<T> *t2, const EvTab &t, int tid)
{
    using F = EvenFFT<T, LOGM>;
    for (int i = tid; i < F::T2; i += ev_threads<T, LOGM>()) t2[i] = ((const cx<T> *)t.t)[F::T1 + i];
}

// P1: each line is one row ky <= nky / 2 at two consecutive energies, A(e_j) +
// i A(e_j + d) (one band value then serves both).  A block takes LR rows at LP
// pairs of energies side by side and walks jc times on; the lines of a row read
// the same band values through the L1 (held in registers they would cost the
// block its partner on the CU).  The result rows leave through LDS in 16-byte
// pieces of the tiles; the blocks whose rows share 128-byte lines run on one
// XCD.
template <typename T, int LOGM, bool W>
__global__ void __launch_bounds__((ev_threads<T, LOGM>()), (sizeof(T) == 4 ? 6 : 3))
    k_be1(const double *__restrict__ xi, Geo g, double emin, double deps, double gamma, EvTab tx, T *__restrict__ spec,
          const T *__restrict__ rho, int jc)
{
    using F = EvenFFT<T, LOGM>;
    constexpr int L = ev_lines<T, LOGM>(), NT = ev_threads<T, LOGM>(), LS = ev_stride<T, LOGM>(false);
    constexpr int LP = kEvPairs, LR = L / LP;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem_raw), *t2 = lds + L * LS;
    const int tid = threadIdx.x, line = tid / F::TL, q = tid % F::TL;
    const bool act = q <= F::P / 2;
    const int ky0 = xcd_group(blockIdx.x, LR < 4 ? 4 / LR : 1) * LR, ky = min(ky0 + line / LP, g.Hy - 1);
    if (ky0 >= g.Hy) return;  // padding block (block-uniform)
    const int H = g.nkx / 2;
    ev_fill_t2<T, LOGM>(t2, tx, tid);
    const T gp = (T)(gamma / kPi), g2 = (T)(gamma * gamma);
    const int jbeg = g.jA + 2 * LP * jc * (int)blockIdx.y, jend = min(g.jB, jbeg + 2 * LP * jc);
    constexpr int VEC = 16 / sizeof(T);
    const int items = g.NTe * 2 * L;
    for (int j0 = jbeg; j0 < jend; j0 += 2 * LP) {
        const int qo = q + opaque_zero(), j = j0 + 2 * (line % LP);
        const double ea = emin + (j + 0.5) * deps, eb = emin + (j + 1.5) * deps;
        cx<T> x[kNz];
#pragma unroll
        for (int i = 0; i < kNz; ++i) {
            const int n = ev_index<F::P>(i, qo);
            const bool in = act && n <= H;
            const unsigned o = (unsigned)(ky * g.nkx) + (in ? n : 0);
            const double xb = *at32(xi, o);
            cx<T> w = ev_chirp<T>(tx, n, in);
            if constexpr (W) w = cscale(w, *at32(rho, o));
            x[i] = cmul(mk<T>(lorentz((T)(ea - xb), gp, g2), lorentz((T)(eb - xb), gp, g2)), w);
        }
        ev_convolve<T, LOGM, true>(x, lds + line * LS, lds + line * LS, t2, tx, qo, act, qo);
        __syncthreads();
        if (act) {
#pragma unroll
            for (int i = 0; i < kNz; ++i) {
                const int n = ev_index<F::P>(i, q);
                if (n <= H) lds[line * LS + n] = x[i];
            }
        }
        __syncthreads();
        for (int it = tid + opaque_zero(); it < items; it += NT) {
            const int h = it & 1, r = (it >> 1) % L, tile = (it >> 1) / L;
            const int row = ky0 + r / LP, ja = j0 + 2 * (r % LP);
            if (row >= g.Hy || ja >= jend) continue;
            const int n0 = tile * g.Ce + h * VEC;
            Vec16<T> a, b;
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                const cx<T> z = n0 + i <= H ? lds[r * LS + n0 + i] : mk<T>((T)0, (T)0);
                a.v[i] = z.x;
                b.v[i] = z.y;
            }
            T *da = spec + (size_t)(ja - g.jA) * g.slice_e + (size_t)((tile * g.HyS + row) * g.Ce + h * VEC);
            *reinterpret_cast<lh_u4 *>(da) = __builtin_bit_cast(lh_u4, a);
            if (ja + 1 < jend) *reinterpret_cast<lh_u4 *>(da + g.slice_e) = __builtin_bit_cast(lh_u4, b);
        }
        __syncthreads();
    }
}

// P2 and P4: each line is a pair of neighbouring real columns of a tile (one
// complex value per row), the lines of a tile interleaved lane by lane so that
// a wave's loads and stores cover whole tile rows.  In place, one slice at a
// time for sj slices, streamed past the L1, which holds the tables (2.96 -> 2.47
// ms at 2049^2 x 512).  upper: only the rows ry >= Ce tile are stored (the forward
// pass with the exchange symmetry).  The padding columns (rx > nkx / 2) need no mask
// here: there is one band, and its builder writes them as zeros in every call.
template <typename T, int LOGM>
__global__ void __launch_bounds__((ev_threads<T, LOGM>()), (sizeof(T) == 4 ? 6 : 3))
    k_becol(T *__restrict__ spec, Geo g, EvTab ty, int nslices, int sj, int upper)
{
    using F = EvenFFT<T, LOGM>;
    constexpr int L = ev_lines<T, LOGM>(), LS = ev_stride<T, LOGM>(true), C = 16 / sizeof(T);
    static_assert(L % C == 0, "whole tiles");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem_raw), *t2 = lds + L * LS;
    const int tid = threadIdx.x;
    const int line = tid % L, q = tid / L;                 // first pass
    const int line2 = tid / F::TL, q2 = tid % F::TL;       // length-P transforms
    const int tile = blockIdx.x * (L / C) + line / C, c = line % C;
    const bool act = q <= F::P / 2 && tile < g.NTe;
    const int H = g.nky / 2, nlo = upper ? tile * g.Ce : 0;
    ev_fill_t2<T, LOGM>(t2, ty, tid);
    const int s0 = blockIdx.y * sj, s1 = min(nslices, s0 + sj);
    for (int s = s0; s < s1; ++s) {
        const int z = opaque_zero(), qo = q + z;
        cx<T> *base = reinterpret_cast<cx<T> *>(spec + (size_t)s * g.slice_e);
        const unsigned o0 = (unsigned)((act ? tile : 0) * g.HyS * C + c);
        cx<T> x[kNz];
#pragma unroll
        for (int i = 0; i < kNz; ++i) {
            const int n = ev_index<F::P>(i, qo);
            const bool in = act && n <= H;
            x[i] = cmul(load_nt(at32(base, o0 + (in ? n : 0) * C)), ev_chirp<T>(ty, n, in));
        }
        ev_convolve<T, LOGM>(x, lds + line * LS, lds + line2 * LS, t2, ty, qo, act, q2 + z);
        if (act) {
#pragma unroll
            for (int i = 0; i < kNz; ++i) {
                const int n = ev_index<F::P>(i, qo);
                if (n <= H && n >= nlo) store_nt(at32(base, o0 + n * C), x[i]);
            }
        }
        __syncthreads();
    }
}

// P5: each line holds two rows qy = 2p, 2p + 1 <= nky / 2 of one plane
// (wa S[a] + wb S[b] for an omega between two lags), read through LDS in
// 16-byte pieces.  The result rows C(qx), qx = 0 .. H, are the output rows qy and
// nky - qy at columns qx and nkx - qx, scaled and written Gamma-centred into
// every zone image, times the orbital |M(Q)|^2 if ff (MODE 0); MODE 1 (the RPA
// path) writes the first-zone map of window slot `plane`.  blockIdx.z: the block's
// share of the zone images (see pass_t).
template <typename T, int LOGM, int MODE>
__global__ void __launch_bounds__((ev_threads<T, LOGM>()), (sizeof(T) == 4 ? 6 : 3))
    k_be5(const T *__restrict__ spec, Geo g, EvTab tx, const PlaneSrc *__restrict__ psrc, double scale,
          T *__restrict__ out, int zx, int zy, int ff, double ffs, const double2 *__restrict__ ffx,
          const double2 *__restrict__ ffy)
{
    using F = EvenFFT<T, LOGM>;
    constexpr int L = ev_lines<T, LOGM>(), NT = ev_threads<T, LOGM>(), LS = ev_stride<T, LOGM>(false);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem_raw), *t2 = lds + L * LS;
    T *stage = reinterpret_cast<T *>(smem_raw);  // [2 L][H + 1]
    const int tid = threadIdx.x, line = tid / F::TL, q = tid % F::TL;
    const bool act = q <= F::P / 2;
    const int nkx = g.nkx, nky = g.nky, H = nkx / 2, SW = H + 1, Hy = g.Hy;
    const int plane = blockIdx.y, row0 = blockIdx.x * 2 * L;
    const PlaneSrc ps = MODE == 0 ? psrc[plane] : PlaneSrc{plane, -1, 1.0, 0.0};
    const int onx = MODE == 0 ? zx * nkx : nkx, ony = MODE == 0 ? zy * nky : nky;
    // zone images [im0, im1) of nzx columns of images
    const int nzx = MODE == 0 ? zx : 1, nim = MODE == 0 ? zx * zy : 1;
    const int per = (nim + (int)gridDim.z - 1) / (int)gridDim.z;
    const int im0 = (int)blockIdx.z * per, im1 = min(nim, im0 + per), zi0 = im0 / nzx, zj0 = im0 - zi0 * nzx;
    const int sx = MODE == 0 ? (zx * nkx) / 2 % nkx : 0, sy = MODE == 0 ? (zy * nky) / 2 % nky : 0;
    const size_t oplane = (size_t)(MODE == 0 ? plane : g.m_lo + plane) * ony;
    if (MODE == 0 && ps.a < 0) {  // the plane is zero (block-uniform)
        for (int r = 0; r < 2 * L && row0 + r < Hy; ++r)
            for (int mir = 0; mir < 2; ++mir) {
                const int qy = mir ? (nky - (row0 + r)) % nky : row0 + r;
                for (int im = im0, zi = zi0, zj = zj0; im < im1; ++im) {
                    T *orow = out + (oplane + zi * nky + (qy + sy) % nky) * onx + (size_t)zj * nkx;
                    for (int X = tid; X < nkx; X += NT) orow[X] = (T)0;
                    if (++zj == nzx) zj = 0, ++zi;
                }
            }
        return;
    }
    ev_fill_t2<T, LOGM>(t2, tx, tid);
    const T *src = spec + (size_t)ps.a * g.slice_e;
    const bool blend = ps.b >= 0 || ps.wa != 1.0;
    const T *src2 = spec + (size_t)(ps.b >= 0 ? ps.b : ps.a) * g.slice_e;
    const T wa = (T)ps.wa, wb = (T)ps.wb;
    constexpr int VEC = 16 / sizeof(T);
    const int items = g.NTe * 2 * (2 * L);
    for (int it = tid; it < items; it += NT) {
        const int h = it & 1, r = (it >> 1) % (2 * L), tile = (it >> 1) / (2 * L);
        const int qy = row0 + r, n0 = tile * g.Ce + h * VEC;
        const size_t o = ((size_t)tile * g.HyS + min(qy, Hy - 1)) * g.Ce + h * VEC;
        Vec16<T> v = __builtin_bit_cast(Vec16<T>, *reinterpret_cast<const lh_u4 *>(src + o));
        if (blend) {
            const Vec16<T> y = __builtin_bit_cast(Vec16<T>, *reinterpret_cast<const lh_u4 *>(src2 + o));
#pragma unroll
            for (int i = 0; i < VEC; ++i) v.v[i] = wa * v.v[i] + wb * y.v[i];
        }
#pragma unroll
        for (int i = 0; i < VEC; ++i)
            if (n0 + i <= H) stage[r * SW + n0 + i] = qy < Hy ? v.v[i] : (T)0;
    }
    cx<T> x[kNz];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kNz; ++i) {
        const int n = ev_index<F::P>(i, q);
        const bool in = act && n <= H;
        const int m = in ? n : 0;
        x[i] = cmul(mk<T>(stage[2 * line * SW + m], stage[(2 * line + 1) * SW + m]), ev_chirp<T>(tx, n, in));
    }
    __syncthreads();
    ev_convolve<T, LOGM>(x, lds + line * LS, lds + line * LS, t2, tx, q, act, q);
    if (!act) return;
    const T sc = (T)scale;
    for (int half = 0; half < 2; ++half) {
        const int qy0 = row0 + 2 * line + half;
        if (qy0 >= Hy) continue;
        for (int mir = 0; mir < 2; ++mir) {
            const int qy = mir ? (nky - qy0) % nky : qy0;
            if (mir && qy == qy0) continue;
            const int yv = (qy + sy) % nky;
            for (int im = im0, zi = zi0, zj = zj0; im < im1; ++im) {
                const int Y = zi * nky + yv;
                T *orow = out + (oplane + Y) * onx;
                const double2 fy = MODE == 0 && ff ? ffy[Y] : make_double2(1.0, 0.0);
                const int qo = q + opaque_zero();
#pragma unroll
                for (int i = 0; i < kNz; ++i) {
                    const int n = ev_index<F::P>(i, qo);
                    if (n > H) continue;
                    const T val = (half ? x[i].y : x[i].x) * sc;
                    // columns n and nkx - n (the same point when 2 n = 0 or nkx)
                    const int Xa = n + sx, Xb = nkx - n + sx;
                    const int xa = zj * nkx + (Xa >= nkx ? Xa - nkx : Xa);
                    const int xb = zj * nkx + (Xb >= nkx ? Xb - nkx : Xb);
                    if (MODE == 0 && ff) {
                        orow[xa] = (T)((double)val * form_factor_sq(ffx[xa], fy, ffs));
                        if (n > 0 && 2 * n != nkx) orow[xb] = (T)((double)val * form_factor_sq(ffx[xb], fy, ffs));
                    } else {
                        orow[xa] = val;
                        if (n > 0 && 2 * n != nkx) orow[xb] = val;
                    }
                }
                if (++zj == nzx) zj = 0, ++zi;
            }
        }
    }
}

inline unsigned cdiv(long a, long b) { return (unsigned)((a + b - 1) / b); }

EvTab ev_tab(const Plan &pl, bool y)
{
    void *const *t = y ? pl.bsy : pl.bsx;
    return EvTab{t[0], t[1], t[2], y ? pl.g.nky : pl.g.nkx};
}

#define LH_EV_SWITCH(v, CALL)             \
    switch (v) {                          \
    case 8: CALL(8); break;               \
    case 9: CALL(9); break;               \
    case 10: CALL(10); break;             \
    case 11: CALL(11); break;             \
    case 12: CALL(12); break;             \
    default: return hipErrorInvalidValue; \
    }

template <typename T>
hipError_t pass_t(const Plan &pl, int pass, void *out, hipStream_t st)
{
    const Geo &g = pl.g;
    T *spec = (T *)pl.spec;
    if (pass == 1) {
        // enough blocks to fill the chip several times over; the block's band
        // rows, chirps and twiddles are loaded once for its jc energy pairs
        const int pairs = (g.nS + 1) / 2;
#define LH_BE1(LG)                                                                                                   \
    do {                                                                                                             \
        constexpr int L = ev_lines<T, LG>();                                                                         \
        constexpr int LP = kEvPairs, LR = L / LP, GR = LR < 4 ? 4 / LR : 1;                                          \
        const unsigned nx = cdiv(cdiv(g.Hy, LR), 8 * GR) * 8 * GR;                                                   \
        const int jc = (int)std::max(1L, std::min(8L, (long)nx * pairs / LP / 2048));                                \
        const auto k = pl.rho ? &k_be1<T, LG, true> : &k_be1<T, LG, false>;                                          \
        hipLaunchKernelGGL(k, dim3(nx, cdiv(pairs, LP * jc)), dim3(ev_threads<T, LG>()), (ev_lds<T, LG>(false)), st, \
                           pl.xi, g, pl.p.emin, pl.deps, pl.p.gamma, ev_tab(pl, false), spec, (const T *)pl.rho, jc); \
    } while (0)
        LH_EV_SWITCH(g.logMx, LH_BE1)
#undef LH_BE1
    } else if (pass == 2 || pass == 4) {
        const int n = pass == 2 ? g.nS : g.nL;
#define LH_BEC(LG)                                                                                                   \
    do {                                                                                                             \
        constexpr int TB = ev_lines<T, LG>() / (16 / (int)sizeof(T));                                                \
        const unsigned nx = cdiv(g.NTe, TB);                                                                         \
        const int sj = (int)std::max(1L, std::min(4L, (long)nx * n / 2048));                                         \
        hipLaunchKernelGGL((k_becol<T, LG>), dim3(nx, cdiv(n, sj)), dim3(ev_threads<T, LG>()), (ev_lds<T, LG>(true)), \
                           st, spec, g, ev_tab(pl, true), n, sj, pass == 2 && g.sw);                                 \
    } while (0)
        LH_EV_SWITCH(g.logMy, LH_BEC)
#undef LH_BEC
    } else {
        const int ff = pl.p.ff_kind != LINDHARD_FF_NONE;
        // a block writes the zone images of its rows one after another (5 to 15 us each,
        // the transform 10): they are dealt out to blocks that repeat the transform, up to
        // 2048 blocks.  257^2 with the orbital, FP32, us a call: 5 x 5 zones x 1 omega 430 ->
        // 67, x 50 omegas 452 -> 246 (with 512 blocks 289, 8192 279); 9 x 9 x 50
        // 1585 -> 643 (889, 598), FP64 1977 -> 1536 (1886, 1478)
        auto images = [&](unsigned nx) {
            const long want = 2048 / std::max(1L, (long)nx * pl.p.nomega);
            return (unsigned)std::max(1L, std::min({want, (long)pl.zx * pl.zy, 65535L}));
        };
#define LH_BE5(LG)                                                                                                   \
    do {                                                                                                             \
        constexpr int L = ev_lines<T, LG>();                                                                         \
        const unsigned nx = cdiv(g.Hy, 2 * L);                                                                       \
        if (pl.p.want_rpa)                                                                                           \
            hipLaunchKernelGGL((k_be5<T, LG, 1>), dim3(nx, g.nL), dim3(ev_threads<T, LG>()), (ev_lds<T, LG>(false)), st, \
                               spec, g, ev_tab(pl, false), pl.d_src, pl.scale, (T *)pl.im1, 1, 1, 0, 0.0, pl.ffx,    \
                               pl.ffy);                                                                              \
        else                                                                                                         \
            hipLaunchKernelGGL((k_be5<T, LG, 0>), dim3(nx, pl.p.nomega, images(nx)), dim3(ev_threads<T, LG>()),      \
                               (ev_lds<T, LG>(false)), st, spec, g, ev_tab(pl, false), pl.d_src, pl.scale, (T *)out, \
                               pl.zx, pl.zy, ff, pl.ff_s, pl.ffx, pl.ffy);                                           \
    } while (0)
        LH_EV_SWITCH(g.logMx, LH_BE5)
#undef LH_BE5
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_even_any(const Plan &pl, int pass, void *out, hipStream_t st)
{
    return pl.g.fp64 ? pass_t<double>(pl, pass, out, st) : pass_t<float>(pl, pass, out, st);
}

// Order of a chirp spectrum (H[0 .. 2^logM)) and twiddles as EvenFFT reads them.
size_t even_any_spectrum_len(int logM) { return (size_t)9 << (logM - 4); }
size_t even_any_spectrum_index(int logM, size_t e)
{
    const int R3 = 1 << (logM - 8), TL = 9 * R3;
    const int i = (int)(e / TL), q = (int)(e % TL), k = q / R3, t = q % R3, u = i / R3, k2 = i % R3;
    return (size_t)(k + 16 * (t + R3 * u + 16 * k2));
}
size_t even_any_twiddle_len(int logM) { return 8 * (((size_t)1 << (logM - 5)) + 1) + ((size_t)15 << (logM - 8)); }
// twiddle e is exp(-2 pi i x / 2^logM) with this x
size_t even_any_twiddle_index(int logM, size_t e)
{
    const size_t G = ((size_t)1 << (logM - 5)) + 1, R3 = (size_t)1 << (logM - 8);
    if (e < 8 * G) return (e / G + 1) * (e % G);
    e -= 8 * G;
    return 16 * (e / R3 + 1) * (e % R3);
}

}  // namespace lh

// lh_maps.hip -- the extended output maps of the RPA path: Im chi from the
// first-zone planes (k_map<..., false>), and Re chi, Im / Re chi_RPA,
// chi_RPA = chi / (1 - V chi) with chi = |M|^2 (Re + i Im) and a contact (vkind 0)
// or Coulomb (vkind 1) interaction, FP64 arithmetic, rounded once to T
// (k_map<..., true>).
//
// Bound by the writes: every first-zone value is read once per row of zones and
// written to each zone.  A thread holds 16 bytes of consecutive columns of one
// output row in up to ZC zones, with the form factors (and Coulomb interactions)
// of all of them in registers, and goes over up to wb omegas; so a block writes whole
// output rows of one plane at a time (10 KB pieces at 512 points and five zones),
// and the zone rows zi of one first-zone row are neighbouring blocks, which read
// it while it is in the last-level cache.  512^2 x 5 x 5 zones x 128 omegas, FP32:
// Im 0.82 -> 0.61 ms for 3.4 GB, the three RPA maps 2.14 -> 1.84 ms for 10.1 GB
// (one thread per point and four omegas with 4-byte stores, the zones outermost,
// before).  The same stores without any read take 0.57 and 1.73 ms; the division
// is hidden (2.05 -> 2.03 ms without it).  Rows as the outer loop with the form
// factor read per value: 1.2 ms and 2.0; zone rows kept on one XCD: 0.70 and 1.95;
// plain in place of nontemporal stores, 512^2 x 3 x 3 zones x 64 omegas: the three
// maps 0.41 -> 0.54 ms; the next omega's loads ahead of the stores: 1.88 ms.
#include <algorithm>
#include <type_traits>

#include "lh_device.h"

namespace lh {

namespace {

struct MapArgs {
    int nkx, nky, nkz, zx, zy, out_nx, out_ny, nw, neps;
    const int *lags, *kkslot;
    const double *fracs;
    int ff, kzn;
    double ffs, V;
    const double2 *ffx, *ffy;
    int logtx, nseg, wb, zc, g0;
};

// VEC consecutive values: one 16-byte access (or one element).
template <typename T, int VEC>
struct MapVec {
    T v[VEC];
};
template <typename T, int VEC>
__device__ __forceinline__ MapVec<T, VEC> map_load(const T *__restrict__ p)
{
    MapVec<T, VEC> r;
    if constexpr (VEC == 1)
        r.v[0] = *p;
    else
        r = __builtin_bit_cast(MapVec<T, VEC>, *reinterpret_cast<const lh_u4 *>(p));
    return r;
}
template <typename T, int VEC>
__device__ __forceinline__ void map_store(T *__restrict__ p, const MapVec<T, VEC> &r)
{
    if constexpr (VEC == 1)
        *p = r.v[0];
    else
        __builtin_nontemporal_store(__builtin_bit_cast(lh_u4, r), reinterpret_cast<lh_u4 *>(p));
}

template <typename T, int VEC, int ZC, bool RPA, bool COUL>
__global__ void __launch_bounds__(256) k_map(const T *__restrict__ im1, const T *__restrict__ re1, MapArgs a,
                                             T *__restrict__ im_out, T *__restrict__ re_out, T *__restrict__ imr,
                                             T *__restrict__ rer)
{
// every form rounds alike, so that a map does not depend on its address
#pragma clang fp contract(off)
    using MV = MapVec<T, VEC>;
    // work item: zone row zi fastest, then the segment of the row, then the group
    // of first-zone rows (kz plane outermost)
    const int it = blockIdx.x;
    const int zi = it % a.zy, rest = it / a.zy, seg = rest % a.nseg;
    const int r = (a.g0 + rest / a.nseg) * (256 >> a.logtx) + ((int)threadIdx.x >> a.logtx);  // row of nkz x nky
    const int xu = ((seg << a.logtx) + (threadIdx.x & ((1 << a.logtx) - 1))) * VEC;  // column within a zone
    if (r >= a.nky * a.nkz || xu >= a.nkx) return;
    const int Zc = r / a.nky, yv = r - Zc * a.nky, zr = a.zy * a.nky, Yb = zi * a.nky + yv, Y = Zc * zr + Yb;
    // the first-zone row it shows
    const int vy = (yv + a.nky - (zr / 2) % a.nky) % a.nky, vz = (Zc + a.nkz - a.nkz / 2) % a.nkz;
    const int u = (xu + a.nkx - ((a.zx * a.nkx) / 2) % a.nkx) % a.nkx;
    const size_t nk = (size_t)a.nkx * a.nky * a.nkz, q = ((size_t)vz * a.nky + vy) * a.nkx + u;
    const size_t plane = (size_t)a.out_nx * a.out_ny;
    const int zj0 = (int)blockIdx.z * a.zc, nz = min(a.zc, a.zx - zj0);  // (nz <= ZC)
    double m2[ZC][VEC], U[ZC][VEC];
    bool qz[ZC][VEC];
#pragma unroll
    for (int z = 0; z < ZC; ++z) {
        if (z >= nz) break;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const int X = (zj0 + z) * a.nkx + xu + i;
            m2[z][i] = a.ff ? form_factor_sq(a.ffx[X], a.ffy[Yb], a.ffs) : 1.0;
            U[z][i] = a.V;
            qz[z][i] = false;
            if constexpr (RPA && COUL) {
                // V / |Q|^2 with Q = 2 pi (h, l, hz) in units of 1/a (h, l the
                // reciprocal-lattice coordinates of X, Y: a grid spanning kzn zones
                // has a step of kzn / n; hz that of the kz plane, lattice constant a
                // along z too); at Q = 0 chi_RPA -> -1/V -> 0
                const double hz = (double)(Zc - a.nkz / 2) / a.nkz;
                const double l = (double)a.kzn * (Yb - zr / 2) / a.nky;
                const double h = (double)a.kzn * (X - (a.zx * a.nkx) / 2) / a.nkx;
                const double q2 = (2.0 * kPi) * (2.0 * kPi) * fma(h, h, fma(l, l, hz * hz));
                qz[z][i] = q2 == 0.0;
                U[z][i] = qz[z][i] ? 0.0 : a.V / q2;
            }
        }
    }
    const int w0 = (int)blockIdx.y * a.wb, w1 = min(w0 + a.wb, a.nw);
    size_t o0 = (size_t)w0 * plane + (size_t)Y * a.out_nx + xu + (size_t)zj0 * a.nkx;
    for (int w = w0; w < w1; ++w, o0 += plane) {
        const int m = a.lags[w];
        const double f = a.fracs[w];
        const bool ina = m >= 1 && m < a.neps, inb = m + 1 >= 1 && m + 1 < a.neps;
        MV im = map_load<T, VEC>(im1 + (size_t)(ina ? m : 1) * nk + q), re;
        if (!ina) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) im.v[i] = (T)0;
        }
        if (f > 0.0) {
            const MV y = map_load<T, VEC>(im1 + (size_t)(inb ? m + 1 : 1) * nk + q);
#pragma unroll
            for (int i = 0; i < VEC; ++i)
                im.v[i] = (T)fma(f, (double)(inb ? y.v[i] : (T)0), (1.0 - f) * (double)im.v[i]);
        }
        if constexpr (RPA) {
            // Re chi at the omega: its lag's plane, or the blend of two lags
            const int sa = a.kkslot[2 * w], sb = a.kkslot[2 * w + 1];
            re = map_load<T, VEC>(re1 + (size_t)sa * nk + q);
            if (f > 0.0 && sb >= 0) {
                const MV y = map_load<T, VEC>(re1 + (size_t)sb * nk + q);
#pragma unroll
                for (int i = 0; i < VEC; ++i) re.v[i] = (T)fma(f, (double)y.v[i], (1.0 - f) * (double)re.v[i]);
            }
        }
#pragma unroll
        for (int z = 0; z < ZC; ++z) {
            if (z >= nz) break;
            MV oi, orr, x = im, r = re;
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                if (a.ff) {
                    x.v[i] = (T)((double)im.v[i] * m2[z][i]);
                    if constexpr (RPA) r.v[i] = (T)((double)re.v[i] * m2[z][i]);
                }
                if constexpr (RPA) {
                    const double xi = (double)x.v[i], ri = (double)r.v[i];
                    const double p = fma(-U[z][i], ri, 1.0), b = U[z][i] * xi;
                    const double inv = 1.0 / fma(p, p, b * b);
                    oi.v[i] = qz[z][i] ? (T)0 : (T)(xi * inv);
                    orr.v[i] = qz[z][i] ? (T)0 : (T)(fma(-b, xi, ri * p) * inv);
                }
            }
            const size_t o = o0 + (size_t)z * a.nkx;
            if constexpr (RPA) {
                if (re_out) map_store<T, VEC>(re_out + o, r);
                if (imr) map_store<T, VEC>(imr + o, oi);
                if (rer) map_store<T, VEC>(rer + o, orr);
            } else {
                map_store<T, VEC>(im_out + o, x);
            }
        }
    }
}

template <typename T>
hipError_t map_t(const Plan &pl, bool rpa, T *im, int vkind, double V, T *re, T *imr, T *rer, hipStream_t st)
{
    const Geo &g = pl.g;
    MapArgs a{};
    a.nkx = g.nkx;
    a.nky = g.nky;
    a.nkz = g.nkz;
    a.zx = pl.zx;
    a.zy = pl.zy;
    a.out_nx = pl.out_nx;
    a.out_ny = pl.out_ny;
    a.nw = pl.p.nomega;
    a.neps = g.neps;
    a.lags = pl.d_lag;
    a.kkslot = pl.d_kkslot;
    a.fracs = pl.d_frac;
    a.ff = pl.p.ff_kind != LINDHARD_FF_NONE;
    a.ffs = pl.ff_s;
    a.ffx = pl.ffx;
    a.ffy = pl.ffy;
    a.V = V;
    a.kzn = pl.p.k_zones;
    // 16-byte accesses: rows of whole vectors, the zone shift too, and aligned outputs
    constexpr int VEC = 16 / sizeof(T);
    auto al = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    const bool vec = g.nkx % (2 * VEC) == 0 && al(im) && al(re) && al(imr) && al(rer);
    const int items = vec ? g.nkx / VEC : g.nkx;
    a.logtx = 4;
    while (a.logtx < 8 && (1 << a.logtx) < items) ++a.logtx;
    a.nseg = (items + (1 << a.logtx) - 1) >> a.logtx;
    // columns of zones in equal groups of up to five; of three while a block goes over
    // at most eight omegas, too few to repay five zones' form factors and registers
    // (a call with RPA, us: 256^2 x 5 x 5 zones x 8 omegas 105 -> 99, 512^2 x 9 x 9 x 1
    // 215 -> 211, x 2 273 -> 267; at 60 omegas 256^2 x 5 x 5 takes 364 with five, 371 with
    // three.  With 11 zones in 5 + 5 + 1: 512^2 x 2 346, in 4 + 4 + 3 336)
    const int gmax = a.nw <= 8 ? 3 : 5;
    const int rpb = 256 >> a.logtx, nz = (pl.zx + gmax - 1) / gmax;
    a.zc = (pl.zx + nz - 1) / nz;
    const int zc = a.zc == 1 ? 1 : a.zc <= 3 ? 3 : 5;
    const int groups = (g.nky * g.nkz + rpb - 1) / rpb, per = a.nseg * pl.zy;  // of rows; blocks of one
    const long nblk = (long)groups * per;
    // omegas per block: 16 for one array and 8 for three (each measured best at
    // 128 omegas: 16 gives 0.61 / 1.89 ms, 8 gives 0.66 / 1.84), fewer while that
    // leaves less than two blocks per CU
    a.wb = rpa ? 8 : 16;
    while (a.wb > 1 && nblk * nz * ((a.nw + a.wb - 1) / a.wb) < 512) a.wb /= 2;
    while ((a.nw + a.wb - 1) / a.wb > 65535) a.wb *= 2;
    // at most 2^19 blocks along x in one launch (a launch takes 2^32 threads there)
    const int gl = std::max(1, (1 << 19) / per);
    const auto go = [&](auto vc, auto zcc) {
        constexpr int VC = decltype(vc)::value, ZC = decltype(zcc)::value;
        const auto k = !rpa ? &k_map<T, VC, ZC, false, false>
                            : vkind == 1 ? &k_map<T, VC, ZC, true, true> : &k_map<T, VC, ZC, true, false>;
        for (a.g0 = 0; a.g0 < groups; a.g0 += gl) {
            const dim3 grid(std::min(gl, groups - a.g0) * per, (a.nw + a.wb - 1) / a.wb, nz);
            hipLaunchKernelGGL(k, grid, dim3(256), 0, st, (const T *)pl.im1, (const T *)pl.re1, a, im, re, imr, rer);
        }
    };
    using I1 = std::integral_constant<int, 1>;
    using I3 = std::integral_constant<int, 3>;
    using I5 = std::integral_constant<int, 5>;
    using IV = std::integral_constant<int, VEC>;
    if (vec)
        zc == 1 ? go(IV{}, I1{}) : zc == 3 ? go(IV{}, I3{}) : go(IV{}, I5{});
    else
        zc == 1 ? go(I1{}, I1{}) : zc == 3 ? go(I1{}, I3{}) : go(I1{}, I5{});
    return hipGetLastError();
}

}  // namespace

hipError_t launch_extend(const Plan &pl, void *out, hipStream_t st)
{
    return pl.g.fp64 ? map_t<double>(pl, false, (double *)out, 0, 0.0, nullptr, nullptr, nullptr, st)
                     : map_t<float>(pl, false, (float *)out, 0, 0.0, nullptr, nullptr, nullptr, st);
}
hipError_t launch_rpa_map(const Plan &pl, int vkind, double V, void *re, void *imr, void *rer, hipStream_t st)
{
    return pl.g.fp64
               ? map_t<double>(pl, true, nullptr, vkind, V, (double *)re, (double *)imr, (double *)rer, st)
               : map_t<float>(pl, true, nullptr, vkind, V, (float *)re, (float *)imr, (float *)rer, st);
}

}  // namespace lh

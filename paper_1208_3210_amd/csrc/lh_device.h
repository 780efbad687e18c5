// lh_device.h -- small device helpers shared by the kernel sources.
#pragma once
#include "lh_fft.h"
#include "lh_internal.h"
#include "lh_regfft.h"

namespace lh {

constexpr double kPi = 3.14159265358979323846;

// 16 bytes of consecutive elements (one vector load or store per lane).
template <typename T>
struct Vec16 {
    T v[16 / sizeof(T)];
};
typedef unsigned lh_u4 __attribute__((ext_vector_type(4)));

// Lorentzian of Eq. (5) from the (already rounded) argument d = e_j - xi_k:
// (gamma/pi) / (d^2 + gamma^2).  FP32 uses the hardware reciprocal (1 ulp).
__device__ __forceinline__ float lorentz(float d, float gp, float g2)
{
    return gp * __builtin_amdgcn_rcpf(d * d + g2);
}
__device__ __forceinline__ double lorentz(double d, double gp, double g2) { return gp / (d * d + g2); }

// |M(Q)|^2 = F(Q)^2 at extended (X, Y), Eq. (3) for the Gaussian d orbital (rounded
// alike in every kernel: no contraction left to the compiler).
__device__ __forceinline__ double form_factor_sq(const double2 fx, const double2 fy, double s)
{
#pragma clang fp contract(off)
    const double q2 = fx.y + fy.y;
    const double dq = fx.y - fy.y;
    const double F = fx.x * fy.x * fma(s * s * dq, dq, fma(-2.0 * s, q2, 1.0));
    return F * F;
}

// Store past the caches (NT) or a plain one.  The last row passes store their maps past
// the caches, which then keep the spectra that the pass reads, from rows of 1024
// points on (two bands 1024^2 x 129 lags: 171 -> 144 us for the pass, 2048^2 x 256 FP64:
// 2.20 -> 2.14 ms, 1024 x 512 x 128 with a caller's band: 130 -> 117; at 512^2 x 64 a
// call takes 93 and 95 us, at 256^2 x 64 with 3 x 3 zones 69 and 94).  Not the pair maps,
// which the next pair reads back (1024^2 x 16 lags x 4 pairs, a call 559 -> 528 us).
// Builder and column passes store large spectra so (se_past).
template <bool NT, typename T>
__device__ __forceinline__ void store_past(T *p, T v)
{
    if constexpr (!NT) {
        *p = v;
    } else {
        typedef unsigned nt_bits __attribute__((ext_vector_type(sizeof(T) / 4)));
        __builtin_nontemporal_store(__builtin_bit_cast(nt_bits, v), reinterpret_cast<nt_bits *>(p));
    }
}

// A zero the optimiser cannot see through.  Added to a thread's position in
// a loop body it keeps the loads and LDS addresses that depend on it inside
// the loop, rather than hoisted out and held in registers across it.
__device__ __forceinline__ int opaque_zero()
{
    int z = 0;
    asm volatile("" : "+s"(z));
    return z;
}

// Launch index -> work index such that grp consecutive work items (which
// share cache lines) run on one XCD: blocks are dispatched round-robin over the
// 8 XCDs, launch index b on XCD b mod 8.  The grid is padded to a multiple of
// 8 grp blocks; the caller skips work indices past its range.
__device__ __forceinline__ int xcd_group(int b, int grp)
{
    const int xcd = b & 7, i = b >> 3;
    return ((i / grp) * 8 + xcd) * grp + i % grp;
}

// Where a run of the window's points lies: element offset p in the slice, and
// with the exchange symmetry (g.sw) the tile t and row r of the first point.
struct WinRun {
    size_t p;
    int t, r;
};
// Points a window pass runs on.
__host__ __device__ __forceinline__ size_t win_points(const Geo &g)
{
    return g.sw ? (size_t)g.sw_units * 4 * g.Ce : g.slice_e;
}
// The run that starts at point i (runs of a power of two of at most 4 Ce points
// that start at a multiple of their length do not leave one unit).
__device__ __forceinline__ WinRun win_run(const Geo &g, size_t i)
{
    if (!g.sw) return WinRun{i, 0, 0};
    // unit u -> tile t: the units before tile t are A t - c t (t - 1) / 2
    const int ue = 4 * g.Ce, u = (int)(i / ue), e = (int)(i % ue), A = g.sw_A, c = g.Ce / 4;
    auto base = [&](int t) { return A * t - c * (t * (t - 1) / 2); };
    const float b = (float)(2 * A + c);
    int t = (int)((b - sqrtf(fmaxf(b * b - 8.0f * c * (float)u, 0.0f))) / (float)(2 * c));
    t = min(max(t, 0), g.NTe - 1);
    while (t + 1 < g.NTe && base(t + 1) <= u) ++t;
    while (t > 0 && base(t) > u) --t;
    const int r = g.Ce * t + 4 * (u - base(t)) + e / g.Ce;
    return WinRun{((size_t)t * g.HyS + r) * g.Ce + e % g.Ce, t, r};
}
// Element offset of the exchanged point of (tile t, row r, column c of the
// tile), or -1 where there is none to write (the tile's own diagonal block holds
// both; padding).
__device__ __forceinline__ long win_mirror(const Geo &g, int t, int r, int c)
{
    const int rx = t * g.Ce + c, t2 = r >> g.logCe;
    if (!g.sw || t2 <= t || rx > g.L || r >= g.Hy) return -1;
    return ((long)t2 * g.HyS + rx) * g.Ce + (r & (g.Ce - 1));
}

// FP32: an FFT twiddle table of n values copied into LDS at dst (stored with
// tw_swz), so that the transform passes read it there rather than waiting on
// the cache for every pass; returns the table to use.  FP64 keeps the global table (it would
// double the LDS of the blocks that use it).  Every thread of the block calls
// it (it ends with a barrier when it copies).
template <typename T>
constexpr bool kTwLds = sizeof(T) == 4;  // the kernels that copy their twiddles into LDS (FP32)
template <typename T>
__device__ __forceinline__ const cx<T> *tw_to_lds(const cx<T> *tw, cx<T> *dst, int n, int tid, int nthr)
{
    if constexpr (kTwLds<T>) {
        for (int i = tid; i < n; i += nthr) dst[tw_swz(i)] = tw[i];  // the layout RegFFT<..., true> reads
        __syncthreads();
        return dst;
    } else {
        return tw;
    }
}
// LDS bytes of such a table
template <typename T>
constexpr size_t tw_lds_bytes(int n)
{
    return sizeof(T) == 4 ? (size_t)n * sizeof(cx<T>) : 0;
}

// Blocks are dispatched round-robin over the 8 XCDs (each with its own L2).
// Map launch index b to a logical tile so that consecutive logical tiles run
// on the same XCD: tiles sharing cache lines then meet in the same L2.
__device__ __forceinline__ unsigned xcd_tile(unsigned b, unsigned nblocks)
{
    const unsigned per = nblocks >> 3;          // full rounds of 8
    if (b >= (per << 3)) return b;              // ragged tail keeps its index
    return (b & 7) * per + (b >> 3);
}

// LDS written by some lanes of a wave is read by others of the same wave: the
// LDS serves one wave's accesses in order, so only the compiler has to keep
// them so.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Element i of an array below 4 GiB: a uniform base plus a 32-bit byte offset
// (one address register per lane instead of two).
template <typename T>
__device__ __forceinline__ T *at32(T *p, unsigned i)
{
    return reinterpret_cast<T *>(reinterpret_cast<char *>(p) + i * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ const T *at32(const T *p, unsigned i)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(p) + i * (unsigned)sizeof(T));
}

}  // namespace lh

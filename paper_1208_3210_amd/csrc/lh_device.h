// lh_device.h -- small device helpers shared by the kernel sources.
#pragma once
#include "lh_fft.h"
#include "lh_internal.h"

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

// |M(Q)|^2 = F(Q)^2 at extended (X, Y), Eq. (3) for the Gaussian d orbital.
__device__ __forceinline__ double form_factor_sq(const double2 fx, const double2 fy, double s)
{
    const double q2 = fx.y + fy.y;
    const double dq = fx.y - fy.y;
    const double F = fx.x * fy.x * (1.0 - 2.0 * s * q2 + s * s * dq * dq);
    return F * F;
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

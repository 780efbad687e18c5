// lh_energy_fft.hip -- energy window of the general path by FFT along the energy
// axis.
#include <algorithm>

#include "lh_device.h"

namespace lh {

namespace {

// S(r, m) = sum_j conj(P_j) H_{j+m} for one real-space point, P_j = B(r, j) for
// occupied j and H_j for unoccupied j (zero elsewhere).  Because every occupied
// index lies below every unoccupied one, the circular correlation of length N >=
// (number of slices) equals the linear one for 0 <= m < N, so
//   S(r, m) = IFFT_N( conj(FFT_N P) * FFT_N H )(m) / N.
// One block: TR real-space points (whole rows of one column tile), G threads per
// point, thread gg with the energies gg + s G in registers, loaded straight from
// the slices (consecutive lanes hold consecutive points of one slice) and stored
// in place in the same pattern.
//
// 2.1 million points x 512 energies x 256 lags (FP32, three dimensions): 6.17 ms
// with the values staged through LDS, whole-length transforms and blocks in tile
// order; 5.4 with the loads straight to registers, the zero halves left out and
// the padded engine; 4.3 (3.0 TB/s) with neighbouring runs on one XCD.  262
// thousand points x 256 x 128: 0.49 -> 0.37 ms.  Bound by HBM latency: each block
// reads one 64- or 128-byte piece of every slice.
//
// HALF: at most N / 2 occupied and N / 2 unoccupied slices.  P is shifted up to
// end at N / 2 and H starts there (the correlation does not see the shift), so P
// sits in the values s < E / 2 and H in the others: the first pass leaves out its
// zero half, and a thread holds one value per s until the transforms run.  LOW:
// only lags m <= N / 2 are wanted, the values s < E / 2 and N / 2 itself.
// Transform engine: the padded one from 64 energies on (lines of G threads,
// padding every min(G, 32) values: an exchange address is a base plus a constant;
// with the swizzled one 512 energies take more than 128 registers and spill under
// that bound), else the swizzled one.
template <int LOGN>
constexpr bool kPadded = LOGN >= 6;
template <typename T, int LOGN, bool INV, unsigned NZ>
struct EngineOf {
    static constexpr int PB = LOGN - 4 < 5 ? LOGN - 4 : 5;
    using P = RegFFTP<T, LOGN, INV, 4, PB, NZ>;
};
// LDS values between lines (interleaved lane by lane: line starts 32 / TR slots
// apart modulo 32)
template <typename T, int LOGN>
__host__ __device__ constexpr int line_stride(int TR)
{
    if constexpr (kPadded<LOGN>) {
        const int L = EngineOf<T, LOGN, false, 0xFFFFFFFFu>::P::LINE, want = TR < 32 ? 32 / TR : 1;
        return L + ((want - L) % 32 + 32) % 32;
    } else {
        return 1 << LOGN;
    }
}
template <typename T, int LOGN>
constexpr size_t lds_bytes(int TR)
{
    if constexpr (kPadded<LOGN>)
        return (size_t)(TR * line_stride<T, LOGN>(TR) + EngineOf<T, LOGN, false, 0xFFFFFFFFu>::P::TWN) * sizeof(cx<T>);
    else
        return ((size_t)TR << LOGN) * sizeof(cx<T>) + tw_lds_bytes<T>(1 << LOGN);
}
template <typename T, int LOGN, bool INV, unsigned NZ>
__device__ __forceinline__ void transform(cx<T> *v, cx<T> *buf, const cx<T> *tw, int gg, int lx)
{
    if constexpr (kPadded<LOGN>)
        EngineOf<T, LOGN, INV, NZ>::P::run(v, buf, tw, gg);
    else
        RegFFT<T, LOGN, INV, 4, kTwLds<T>, NZ>::run(v, buf, tw, 0, gg, lx);
}
// Threads of a block: up to 256 (512 for 2048 energies in FP32, 128 threads a line)
template <int LOGN>
constexpr int kMaxThreads = LOGN >= 11 ? 512 : 256;

template <typename T, int LOGN, bool HALF, bool LOW>
__global__ void __launch_bounds__(kMaxThreads<LOGN>, sizeof(T) == 4 ? (LOGN >= 9 ? 3 : 4) : 1)
    k_p3f(cx<T> *__restrict__ spec, Geo g, const cx<T> *__restrict__ twe)
{
    using F = RegFFT<T, LOGN, false>;
    constexpr int N = F::N, E = F::E, G = F::G;
    constexpr unsigned LO = (1u << (E / 2)) - 1, ALL = 0xFFFFFFFFu;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cx<T> *lds = reinterpret_cast<cx<T> *>(smem_raw);  // [TR][line stride], the twiddles
    const int TR = g.p3f_TR, logTR = g.p3f_logTR, LS = line_stride<T, LOGN>(TR);
    const int tid = threadIdx.x;
    const int rp = tid & (TR - 1), gg = tid >> logTR;
    // consecutive runs of points on one XCD: their 128-byte pieces of a slice are
    // neighbours
    const size_t off = (size_t)xcd_tile(blockIdx.x, gridDim.x) * TR + rp;
    const int ne = g.nS, j0 = g.j0 - g.jA;
    const cx<T> zero = mk<T>((T)0, (T)0);
    const cx<T> *tw;
    if constexpr (kPadded<LOGN>) {
        EngineOf<T, LOGN, false, ALL>::P::fill_twiddles(lds + TR * LS, twe, tid, TR * G);
        tw = lds + TR * LS;
        // (read first in the second pass, after the first exchange's barrier)
    } else {
        tw = tw_to_lds<T>(twe, lds + TR * LS, N, tid, TR * G);
    }
    cx<T> vp[E], vh[E];
    if constexpr (HALF) {
        const int sh = N / 2 - j0;  // place of slice j: j + sh
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = gg + s * G - sh;
            const bool in = j >= 0 && j < ne;
            const cx<T> b = spec[(size_t)(in ? j : 0) * g.slice_elems + off];
            (s < E / 2 ? vp : vh)[s] = in ? b : zero;
        }
    } else {
#pragma unroll
        for (int s = 0; s < E; ++s) {
            const int j = gg + s * G;
            const cx<T> b = spec[(size_t)(j < ne ? j : 0) * g.slice_elems + off];
            vp[s] = j < j0 ? b : zero;
            vh[s] = j >= j0 && j < ne ? b : zero;
        }
    }
    cx<T> *buf = lds + rp * LS;
    const int lxe = lds_xor_interleaved<T, N>(rp, TR);
    transform<T, LOGN, false, HALF ? LO : ALL>(vp, buf, tw, gg, lxe);
    transform<T, LOGN, false, HALF ? LO << (E / 2) : ALL>(vh, buf, tw, gg, lxe);
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const cx<T> a = vp[s], b = vh[s];
        vh[s] = mk<T>(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);  // conj(a) b
    }
    transform<T, LOGN, true, ALL>(vh, buf, tw, gg, lxe);
    const T inv = (T)(1.0 / N);
#pragma unroll
    for (int s = 0; s < (LOW ? E / 2 + 1 : E); ++s) {
        const int m = gg + s * G;
        if (m >= g.m_lo && m <= g.m_hi) spec[(size_t)(m - g.m_lo) * g.slice_elems + off] = cscale(vh[s], inv);
    }
}

template <typename T, int LOGN>
void launch_t(const Plan &pl, hipStream_t st)
{
    const Geo &g = pl.g;
    using F = RegFFT<T, LOGN, false>;
    const int j0 = g.j0 - g.jA, half = 1 << (LOGN - 1);
    const bool h = F::E >= 2 && j0 <= half && g.nS - j0 <= half, low = h && g.m_hi <= half;
    const auto k = low ? &k_p3f<T, LOGN, true, true> : h ? &k_p3f<T, LOGN, true, false> : &k_p3f<T, LOGN, false, false>;
    hipLaunchKernelGGL(k, dim3((unsigned)(g.slice_elems / g.p3f_TR)), dim3(g.p3f_TR * F::G),
                       (lds_bytes<T, LOGN>(g.p3f_TR)), st, (cx<T> *)pl.spec, g,
                       (const cx<T> *)pl.twe);
}

template <typename T>
hipError_t p3f_t(const Plan &pl, hipStream_t st)
{
#define LH_P3F(LG) case LG: launch_t<T, LG>(pl, st); break
    switch (pl.g.logNE) {
        LH_P3F(1);
        LH_P3F(2);
        LH_P3F(3);
        LH_P3F(4);
        LH_P3F(5);
        LH_P3F(6);
        LH_P3F(7);
        LH_P3F(8);
        LH_P3F(9);
        LH_P3F(10);
        LH_P3F(11);
    default: return hipErrorInvalidValue;
    }
#undef LH_P3F
    return hipGetLastError();
}

}  // namespace

hipError_t launch_p3f(const Plan &pl, hipStream_t st)
{
    return pl.g.fp64 ? p3f_t<double>(pl, st) : p3f_t<float>(pl, st);
}

}  // namespace lh

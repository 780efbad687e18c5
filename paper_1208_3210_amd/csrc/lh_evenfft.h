// lh_evenfft.h -- transform of an even complex sequence on half the work.
//
// The sequences of the mirror-symmetric path are even, z[n] = z[N - n] (two
// real even lines packed as a + i b), so their DFT is even too and the same in
// both directions, Z[j] = sum_n z[n] exp(-+2 pi i n j / N), and half of both is
// redundant.  With N = 16 P, a first pass of radix 16 over n = g + P s needs
// only the butterflies g <= P / 2 (the butterfly of P - g holds the same inputs
// in reverse, so its outputs are those of g), and of the sixteen length-P
// transforms behind it (frequencies j = k + 16 m) only k = 0 .. 8 are needed
// (j -> N - j maps k to 16 - k): 9/16 of the values, exchanges and
// multiplications of a full transform, with no extra rounding step.
//
//   y_g[k]      = sum_s z[g + P s] exp(-2 pi i k s / 16)
//   Y_k[g]      = w^(g k) y_g[k],  Y_k[P - g] = w^(-g k) y_g[16 - k],
//                 w = exp(-2 pi i / N)
//   Z[k + 16 m] = DFT_P(Y_k)[m]
//
// One line is run by TL = 9 P / 16 threads.  In the first pass thread q <= P/2
// has the butterfly g = q; in the length-P transforms thread q = k R3 + t
// (R3 = P / 16 threads for each k) holds 16 values and runs radix 16, then,
// through one more exchange, radix R3.  The inverse runs the steps backwards.
// The thread then holds Z[j(i)], i = u R3 + k2, j = k + 16 (t + R3 u + 16 k2).
//
// LDS of a line: nine rows of PS = P + R3 values; value x of a row sits at
// swz(x) = x ^ ((x / R3) mod R3).  The stride-1 accesses of the first pass, the
// stride-R3 ones of the radix-16 pass and the runs of R3 read by the radix-R3
// pass are then all free of bank conflicts (row starts are R3 apart modulo the
// 32 eight-byte slots), and each exchange inside the length-P transforms reads
// and writes one thread's own set of slots, so it costs one barrier.
#pragma once
#include "lh_device.h"
#include "lh_regfft.h"

namespace lh {

template <typename T, int LOGN>
struct EvenFFT {
    static_assert(LOGN >= 8 && LOGN <= 12, "256 to 4096 points");
    static constexpr int N = 1 << LOGN, P = N / 16, R3 = P / 16, LOGR3 = LOGN - 8;
    static constexpr int TL = 9 * R3;      // threads per line
    static constexpr int PS = P + R3;      // LDS values per row
    static constexpr int LINE = 9 * PS;    // LDS values per line
    static constexpr int Q = 16 / R3;      // radix-R3 butterflies per thread
    // first-pass twiddles w^(g k) at (k - 1) (P / 2 + 1) + g, k = 1 .. 8
    static constexpr int T1 = 8 * (P / 2 + 1);
    // twiddles exp(-2 pi i t s / P) at (s - 1) R3 + t, s = 1 .. 15
    static constexpr int T2 = 15 * R3;

    __device__ static __forceinline__ int swz(int x) { return R3 > 1 ? x ^ ((x >> LOGR3) & (R3 - 1)) : x; }

    // y = the radix-16 DFT of butterfly g (natural order) -> the nine rows at buf
    __device__ static __forceinline__ void split(const cx<T> *y, cx<T> *buf, const cx<T> *__restrict__ t1, int g)
    {
        const int a = swz(g), m = swz((P - g) & (P - 1));
        buf[a] = y[0];
        buf[m] = y[0];
#pragma unroll
        for (int k = 1; k <= 8; ++k) {
            const cx<T> w = *at32(t1, (k - 1) * (P / 2 + 1) + g);
            buf[k * PS + a] = cmul(w, y[k]);
            buf[k * PS + m] = cmul(cconj(w), y[16 - k]);
        }
    }

    // the nine rows -> y, the input of the inverse radix-16 DFT of butterfly g
    __device__ static __forceinline__ void merge(cx<T> *y, const cx<T> *buf, const cx<T> *__restrict__ t1, int g)
    {
        const int a = swz(g), m = swz((P - g) & (P - 1));
        y[0] = buf[a];
#pragma unroll
        for (int k = 1; k <= 8; ++k) {
            const cx<T> w = *at32(t1, (k - 1) * (P / 2 + 1) + g);
            y[k] = cmul(cconj(w), buf[k * PS + a]);
            if (k < 8) y[16 - k] = cmul(w, buf[k * PS + m]);
        }
    }

    // The length-P transform of row `row` by its threads t: v[i] = Z[j(i)].
    // t2: the T2 table (LDS).  A row's threads are lanes of one wave: their exchange
    // takes no block barrier.
    __device__ static __forceinline__ void fwd(cx<T> *v, cx<T> *row, const cx<T> *t2, int t)
    {
#pragma unroll
        for (int s = 0; s < 16; ++s) v[s] = row[s * R3 + (t ^ (s & (R3 - 1)))];
        rdft<T, 16, false>(v);
        if constexpr (R3 > 1) {
#pragma unroll
            for (int s = 0; s < 16; ++s)
                row[s * R3 + (t ^ (s & (R3 - 1)))] = s ? cmul(v[s], t2[(s - 1) * R3 + t]) : v[0];
            wave_sync();
#pragma unroll
            for (int u = 0; u < Q; ++u) {
#pragma unroll
                for (int k = 0; k < R3; ++k) v[u * R3 + k] = row[(t + u * R3) * R3 + (k ^ t)];
                rdft<T, R3, false>(v + u * R3);
            }
        }
    }

    // The inverse of fwd (no 1/P): v[i] = Z[j(i)] -> the row, ready for merge
    // after a barrier.
    __device__ static __forceinline__ void inv(cx<T> *v, cx<T> *row, const cx<T> *t2, int t)
    {
        if constexpr (R3 > 1) {
#pragma unroll
            for (int u = 0; u < Q; ++u) {
                rdft<T, R3, true>(v + u * R3);
#pragma unroll
                for (int k = 0; k < R3; ++k) row[(t + u * R3) * R3 + (k ^ t)] = v[u * R3 + k];
            }
            wave_sync();
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                v[s] = row[s * R3 + (t ^ (s & (R3 - 1)))];
                if (s) v[s] = cmul(v[s], cconj(t2[(s - 1) * R3 + t]));
            }
        }
        rdft<T, 16, true>(v);
#pragma unroll
        for (int s = 0; s < 16; ++s) row[s * R3 + (t ^ (s & (R3 - 1)))] = v[s];
    }
};

}  // namespace lh

// Periodograms of real float64 sequences: |X_k|^2 / len, k = 0 .. len/2.
//
// A real sequence of length len = 2 M is transformed as M complex points
// z_n = x_2n + i x_2n+1 and separated by the Hermitian symmetry at the end, in
// float64 throughout.  Every transform runs in one workgroup: eight points per
// thread in registers, exchanged through LDS between radix-8 Stockham passes
// (a radix-2 or radix-4 pass first where log2 M is not a multiple of three).
//
// len <= 8192: one launch, a workgroup per sequence takes it from the strided
// input to the spectrum (mean, window, transform, separation), so the data
// crosses memory once.  Radix-2 passes through global memory, one launch each,
// took 71 us for 96 sequences of 4096 points (15 launches of 3-5 us); one
// launch takes 12.9 us, call to call, bound by the latency of its passes.
// Error against extended precision, root mean square of the norm over 64 recorded
// sequences: 1.3e-16 to 1.5e-16 at every length from 16 to 65536 samples; the
// radix-2 passes had 1.5e-16 to 2.0e-16.
// Longer: M = M1 x M2; ps_cols transforms the M1-point columns (several
// columns per workgroup, so that the loads stay coalesced) and applies the
// twiddles between the two factors, ps_rows the M2-point rows, ps_separate
// gathers the pairs k and M - k.  M1 = 64 as long as M2 = M / 64 fits one
// workgroup's LDS (4096 points), then 512, then 2048.
#pragma once
#include "llg_device.hpp"

namespace llg {

constexpr int PS_MAX_LOGM = 12;   // points of one workgroup's LDS buffer: 4096 x 16 bytes and padding

__device__ __forceinline__ double2 zadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 zsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 zrot(double2 a) { return make_double2(a.y, -a.x); }   // -i a
// exp(-2 pi i n / d) for 0 <= n < d
__device__ __forceinline__ double2 zroot(long long n, long long d) {
    double s, c;
    sincospi(-2.0 * (double)n / (double)d, &s, &c);
    return make_double2(c, s);
}

template <int R>
__device__ __forceinline__ void zdft(double2* x) {
    if constexpr (R == 2) {
        const double2 t = x[0];
        x[0] = zadd(t, x[1]);
        x[1] = zsub(t, x[1]);
    } else if constexpr (R == 4) {
        const double2 a0 = zadd(x[0], x[2]), a1 = zsub(x[0], x[2]);
        const double2 a2 = zadd(x[1], x[3]), a3 = zrot(zsub(x[1], x[3]));
        x[0] = zadd(a0, a2);
        x[2] = zsub(a0, a2);
        x[1] = zadd(a1, a3);
        x[3] = zsub(a1, a3);
    } else {
        static_assert(R == 8, "radix 2, 4 or 8");
        double2 e[4] = {x[0], x[2], x[4], x[6]}, o[4] = {x[1], x[3], x[5], x[7]};
        zdft<4>(e);
        zdft<4>(o);
        // times sqrt(1/2) with what the constant lacks: its rounding scales a whole line of the spectrum alike
        auto half = [](double v) { return fma(0.70710678118654752440, v, -4.833646656726457e-17 * v); };
        const double2 t1 = make_double2(half(o[1].x + o[1].y), half(o[1].y - o[1].x));
        const double2 t2 = zrot(o[2]);
        const double2 t3 = make_double2(half(o[3].y - o[3].x), -half(o[3].x + o[3].y));
        x[0] = zadd(e[0], o[0]);
        x[4] = zsub(e[0], o[0]);
        x[1] = zadd(e[1], t1);
        x[5] = zsub(e[1], t1);
        x[2] = zadd(e[2], t2);
        x[6] = zsub(e[2], t2);
        x[3] = zadd(e[3], t3);
        x[7] = zsub(e[3], t3);
    }
}

// one padding slot after every 8 points: the writes of a first radix-8 pass
// (stride 8 between threads) and the consecutive reads use all banks
__device__ __forceinline__ int psp(int e) { return e + (e >> 3); }

// Shape of the transforms of one workgroup: NC transforms of 2^LOGM points, one
// after the other in the LDS buffer, PT points per thread.
template <int LOGM, int LOGC>
struct PsShape {
    static constexpr int M = 1 << LOGM, POINTS = M << LOGC;
    static constexpr int THREADS = POINTS / 8 < 64 ? 64 : POINTS / 8;
    static constexpr int LDS = POINTS + POINTS / 8;
};

// Radix-R pass over all transforms of the buffer (sub-transforms of length Ns
// -> R Ns).  Thread t takes the butterflies t, t + threads, ...: at most 8 points.
// v holds the thread's points: butterfly q in v[q R .. q R + R - 1].
template <int LOGM, int LOGC, int R>
__device__ __forceinline__ void ps_load_pass(const double2* buf, double2 (&v)[8]) {
    using S = PsShape<LOGM, LOGC>;
    constexpr int PER = S::M / R, TOTAL = S::POINTS / R;
#pragma unroll
    for (int q = 0; q < 8 / R; ++q) {
        const int b = threadIdx.x + q * S::THREADS;
        if (b >= TOTAL) continue;
        const int c = b / PER, t = b % PER;
#pragma unroll
        for (int j = 0; j < R; ++j) v[q * R + j] = buf[psp(c * S::M + t + j * PER)];
    }
}
template <int LOGM, int LOGC, int R>
__device__ __forceinline__ void ps_store_pass(double2* buf, double2 (&v)[8], int Ns) {
    using S = PsShape<LOGM, LOGC>;
    constexpr int PER = S::M / R, TOTAL = S::POINTS / R;
#pragma unroll
    for (int q = 0; q < 8 / R; ++q) {
        const int b = threadIdx.x + q * S::THREADS;
        if (b >= TOTAL) continue;
        const int c = b / PER, t = b % PER, kk = t & (Ns - 1);
        double2* x = v + q * R;
        // Every factor from the sine.  As a chain of products of the first one (12.9 us for 96 sequences of 8192, 17.4
        // this way; 12.9 both for 4096) they double the spectra's error, and a tree of products does so too; w, w^2
        // and w^4 from the sine and products of those (15.3 us) stay 5 % above the radix-2 passes at some lengths.
        if (Ns > 1)
#pragma unroll
            for (int j = 1; j < R; ++j) x[j] = zmul(x[j], zroot(j * kk, (long long)Ns * R));
        zdft<R>(x);
        const int base = c * S::M + (t - kk) * R + kk;
#pragma unroll
        for (int j = 0; j < R; ++j) buf[psp(base + j * Ns)] = x[j];
    }
}

// The transforms of the buffer, in place.  On entry the first pass's points are
// in v (ps_load_pass of radix PS_FIRST); on exit the buffer holds them in
// natural order behind a workgroup barrier.
template <int LOGM>
constexpr int ps_first_radix() { return LOGM % 3 == 0 ? 8 : 1 << (LOGM % 3); }
template <int LOGM, int LOGC>
__device__ __forceinline__ void ps_transform(double2* buf, double2 (&v)[8]) {
    constexpr int R0 = ps_first_radix<LOGM>();
    ps_store_pass<LOGM, LOGC, R0>(buf, v, 1);
    __syncthreads();
#pragma unroll
    for (int Ns = R0; Ns < (1 << LOGM); Ns *= 8) {
        ps_load_pass<LOGM, LOGC, 8>(buf, v);
        __syncthreads();
        ps_store_pass<LOGM, LOGC, 8>(buf, v, Ns);
        __syncthreads();
    }
}

// Point n of a sequence as the transform takes it: (x_2n, x_2n+1), mean removed, windowed.
__device__ __forceinline__ double2 ps_point(const double* xb, long long n, long long len, long long tstride,
                                            double mean, int window) {
    double2 z = make_double2(xb[2 * n * tstride] - mean, xb[(2 * n + 1) * tstride] - mean);
    if (window == 1) {   // Hann: sin^2(pi t / len)
        const double s0 = sinpi((double)(2 * n) / (double)len), s1 = sinpi((double)(2 * n + 1) / (double)len);
        z.x *= s0 * s0;
        z.y *= s1 * s1;
    }
    return z;
}

// A value with the rounding of the operations that gave it.
struct Exact2 {
    double v, e;
};
__device__ __forceinline__ Exact2 exact_sum(double a, double b) {   // Knuth's two-sum
    const double s = a + b, t = s - a;
    return {s, (a - (s - t)) + (b - t)};
}

// |X_k|^2 / len and |X_M-k|^2 / len from a = Z_k and b = Z_M-k (M = len / 2):
// X_k = E + W O and X_M-k = conj(E - W O) with E = (a + conj b)/2, O = (a - conj b)/(2i), W = exp(-2 pi i k / len).
// The packed transform takes one level of additions more here than a transform
// of the len real samples, and the roundings of the last levels are the ones that
// reach a spectral line undivided; so this one carries them along and rounds once.
__device__ __forceinline__ void ps_pair(double2 a, double2 b, long long k, long long len, double& pk, double& pm) {
#pragma clang fp contract(off)
    const Exact2 Ex = exact_sum(0.5 * a.x, 0.5 * b.x), Ey = exact_sum(0.5 * a.y, -0.5 * b.y);
    const Exact2 Ox = exact_sum(0.5 * a.y, 0.5 * b.y), Oy = exact_sum(0.5 * b.x, -0.5 * a.x);
    const double2 W = zroot(k, len);
    auto add2 = [](Exact2 z, double p, Exact2 x, double q, Exact2 y) {   // z + p x + q y
        const double px = p * x.v, qy = q * y.v;
        const Exact2 s = exact_sum(px, qy), t = exact_sum(z.v, s.v);
        const double e = (fma(p, x.v, -px) + fma(q, y.v, -qy)) + (p * x.e + q * y.e);
        return Exact2{t.v, t.e + (s.e + (z.e + e))};
    };
    auto power = [len](Exact2 x, Exact2 y) {
        const double xx = x.v * x.v, yy = y.v * y.v;
        const Exact2 s = exact_sum(xx, yy);
        if (!isfinite(s.v)) return s.v;
        const double e = (fma(x.v, x.v, -xx) + fma(y.v, y.v, -yy)) + 2.0 * (x.v * x.e + y.v * y.e);
        return (s.v + (s.e + e)) / (double)len;
    };
    pk = power(add2(Ex, W.x, Ox, -W.y, Oy), add2(Ey, W.y, Ox, W.x, Oy));
    pm = power(add2(Ex, -W.x, Ox, W.y, Oy), add2(Ey, -W.y, Ox, -W.x, Oy));
}

// Sum over a workgroup of THREADS threads (every thread gets it).
template <int THREADS>
__device__ __forceinline__ double ps_block_sum(double s, double* sh) {
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) t += sh[w];
    return t;
}

// One sequence of 2^(LOGM + 1) samples per workgroup, from input to spectrum.
template <int LOGM>
__global__ __launch_bounds__((PsShape<LOGM, 0>::THREADS)) void ps_whole(const double* x, long long bstride,
                                                                       long long tstride, int remove_mean, int window,
                                                                       double* out) {
    using S = PsShape<LOGM, 0>;
    constexpr int M = S::M, R0 = ps_first_radix<LOGM>(), PER = M / R0;
    constexpr long long len = 2ll * M;
    __shared__ double2 buf[S::LDS];
    __shared__ double sh[S::THREADS / 64];
    const int b = blockIdx.x;
    const double* xb = x + (long long)b * bstride;
    double2 v[8];
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < 8 / R0; ++q) {
        const int t = threadIdx.x + q * S::THREADS;
        if (t >= PER) continue;
#pragma unroll
        for (int j = 0; j < R0; ++j) {
            v[q * R0 + j] = ps_point(xb, t + j * PER, len, tstride, 0.0, 0);
            sum += v[q * R0 + j].x + v[q * R0 + j].y;
        }
    }
    const double mean = remove_mean ? ps_block_sum<S::THREADS>(sum, sh) / (double)len : 0.0;
#pragma unroll
    for (int q = 0; q < 8 / R0; ++q) {
        const int t = threadIdx.x + q * S::THREADS;
        if (t >= PER) continue;
#pragma unroll
        for (int j = 0; j < R0; ++j) {
            double2& z = v[q * R0 + j];
            z.x -= mean;
            z.y -= mean;
            if (window == 1) {
                const long long n = t + j * PER;
                const double s0 = sinpi((double)(2 * n) / (double)len), s1 = sinpi((double)(2 * n + 1) / (double)len);
                z.x *= s0 * s0;
                z.y *= s1 * s1;
            }
        }
    }
    ps_transform<LOGM, 0>(buf, v);
    double* o = out + (long long)b * (M + 1);
    for (int k = threadIdx.x; k <= M / 2; k += S::THREADS) {
        double pk, pm;
        ps_pair(buf[psp(k)], buf[psp((M - k) & (M - 1))], k, len, pk, pm);
        o[k] = pk;
        o[M - k] = pm;
    }
}

// Spectra from the workspace to a result array that overlaps the input.
__global__ __launch_bounds__(256) void ps_copy(const double* from, long long n, double* to) {
    for (long long q = blockIdx.x * 256ll + threadIdx.x; q < n; q += (long long)gridDim.x * 256) to[q] = from[q];
}

// Mean of each sequence (or 0), for the sequences that take several workgroups.
__global__ __launch_bounds__(1024) void ps_mean(const double* x, long long bstride, long long len, long long tstride,
                                                int remove_mean, double* mean) {
    __shared__ double sh[16];
    const double* xb = x + (long long)blockIdx.x * bstride;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    if (remove_mean)   // len is a power of two beyond 8192: whole rounds of 4096
        for (long long t = threadIdx.x; t < len; t += 4096) {
            s0 += xb[t * tstride];
            s1 += xb[(t + 1024) * tstride];
            s2 += xb[(t + 2048) * tstride];
            s3 += xb[(t + 3072) * tstride];
        }
    const double s = ps_block_sum<1024>((s0 + s1) + (s2 + s3), sh);
    if (threadIdx.x == 0) mean[blockIdx.x] = s / (double)len;
}

// Columns n2 of z (n = n1 M2 + n2): 2^LOGM1-point transforms over n1, 2^LOGC of
// them per workgroup, times exp(-2 pi i n2 k1 / M); to Y[k1 M2 + n2].
template <int LOGM1, int LOGC>
__global__ __launch_bounds__((PsShape<LOGM1, LOGC>::THREADS)) void ps_cols(const double* x, long long bstride,
                                                                          long long len, long long tstride, int window,
                                                                          const double* mean, double2* Y) {
    using S = PsShape<LOGM1, LOGC>;
    constexpr int C = 1 << LOGC;
    __shared__ double2 buf[S::LDS];
    const long long M = len / 2, M2 = M >> LOGM1, n20 = (long long)blockIdx.x * C;
    const double* xb = x + (long long)blockIdx.y * bstride;
    const double mu = mean[blockIdx.y];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int e = threadIdx.x + q * S::THREADS, c = e % C, n1 = e / C;
        buf[psp(c * S::M + n1)] = ps_point(xb, n1 * M2 + n20 + c, len, tstride, mu, window);
    }
    __syncthreads();
    double2 v[8];
    ps_load_pass<LOGM1, LOGC, ps_first_radix<LOGM1>()>(buf, v);
    __syncthreads();
    ps_transform<LOGM1, LOGC>(buf, v);
    double2* yb = Y + (long long)blockIdx.y * M;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int e = threadIdx.x + q * S::THREADS, c = e % C, k1 = e / C;
        const long long n2 = n20 + c;
        yb[k1 * M2 + n2] = zmul(buf[psp(c * S::M + k1)], zroot(n2 * k1, M));
    }
}

// Row k1 of Y: 2^LOGM2-point transform over n2, in place: Z_(k1 + M1 k2) at [k1 M2 + k2].
template <int LOGM2>
__global__ __launch_bounds__((PsShape<LOGM2, 0>::THREADS)) void ps_rows(double2* Y, long long M) {
    using S = PsShape<LOGM2, 0>;
    __shared__ double2 buf[S::LDS];
    double2* row = Y + (long long)blockIdx.y * M + (long long)blockIdx.x * S::M;
    for (int e = threadIdx.x; e < S::M; e += S::THREADS) buf[psp(e)] = row[e];
    __syncthreads();
    double2 v[8];
    ps_load_pass<LOGM2, 0, ps_first_radix<LOGM2>()>(buf, v);
    __syncthreads();
    ps_transform<LOGM2, 0>(buf, v);
    for (int e = threadIdx.x; e < S::M; e += S::THREADS) row[e] = buf[psp(e)];
}

__global__ __launch_bounds__(256) void ps_separate(const double2* Y, long long len, long long M1, double* out) {
    const long long M = len / 2, M2 = M / M1;
    const double2* yb = Y + (long long)blockIdx.y * M;
    double* o = out + (long long)blockIdx.y * (M + 1);
    auto at = [&](long long k) { return yb[(k & (M1 - 1)) * M2 + k / M1]; };
    for (long long k = blockIdx.x * 256ll + threadIdx.x; k <= M / 2; k += (long long)gridDim.x * 256) {
        double pk, pm;
        ps_pair(at(k), at((M - k) & (M - 1)), k, len, pk, pm);
        o[k] = pk;
        o[M - k] = pm;
    }
}

}  // namespace llg

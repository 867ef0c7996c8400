// FP64 Fourier transforms of lines in LDS, any length: mixed-radix Stockham
// passes.  With l the product of the factors taken so far and M = n / l, the
// line holds at k M + q the partial transforms
//     A_l[k][q] = sum_{s < l} x[q + s M] e^{-2 pi i k s / l},
// and a pass with factor P forms, with M' = M / P,
//     A_{lP}[k + l r][q'] = sum_{j < P} e^{-2 pi i r j / P}
//                           (e^{-2 pi i k j / (l P)} A_l[k][q' + j M']).
// Factors 8, 4, 5, 3, 2 are butterflies in registers, one thread each; any
// other prime takes P multiply-adds per output, so a line costs
// n (sum of its prime factors) where a direct transform costs n^2.  A pass
// reads its values, waits, and writes them back in place.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbfss {

constexpr int kFftMaxFactors = 12;
struct FftPlan {
    int32_t n, nf;
    int32_t tmul;  // twiddle table entries per step of e^{-2 pi i / n}
    int32_t f[kFftMaxFactors];
};

// The factors of a transform of n points out of a table of L = n tmul entries.
inline FftPlan fft_plan(int n, int tmul) {
    FftPlan p{};
    p.n = n;
    p.tmul = tmul;
    auto put = [&](int f) { p.f[p.nf++] = f; };
    int m = n, twos = 0;
    while (m % 2 == 0) m /= 2, ++twos;
    for (int f = 3; m > 1; f += 2)
        while (m % f == 0) put(f), m /= f;
    // radix 8, with one or two of radix 4 instead of a radix-2 rest
    if (twos == 1) put(2);
    else {
        const int fours = twos % 3 == 2 ? 1 : (twos % 3 == 1 ? 2 : 0);
        for (int k = 0; k < (twos - 2 * fours) / 3; ++k) put(8);
        for (int k = 0; k < fours; ++k) put(4);
    }
    return p;
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmuli(double2 a) { return make_double2(a.y, -a.x); }  // -i a

// i / d for 0 <= i < 2^21, rd = 1 / d to an ulp
__device__ __forceinline__ int div_small(int i, float rd) { return (int)(((float)i + 0.5f) * rd); }

// the P-point transform of v, in place
template <int P>
__device__ __forceinline__ void dft_point(double2 (&v)[P]) {
    if constexpr (P == 2) {
        const double2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (P == 3) {
        const double s3 = 0.86602540378443864676;
        const double2 s = cadd(v[1], v[2]), d = cmuli(csub(v[1], v[2]));
        const double2 a = make_double2(v[0].x - 0.5 * s.x, v[0].y - 0.5 * s.y);
        v[0] = cadd(v[0], s);
        v[1] = make_double2(a.x + s3 * d.x, a.y + s3 * d.y);
        v[2] = make_double2(a.x - s3 * d.x, a.y - s3 * d.y);
    } else if constexpr (P == 4) {
        const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]), c = cadd(v[1], v[3]), d = cmuli(csub(v[1], v[3]));
        v[0] = cadd(a, c);
        v[1] = cadd(b, d);
        v[2] = csub(a, c);
        v[3] = csub(b, d);
    } else if constexpr (P == 5) {
        const double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;
        const double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;
        const double2 t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]), t3 = csub(v[1], v[4]), t4 = csub(v[2], v[3]);
        const double2 a1 = make_double2(v[0].x + c1 * t1.x + c2 * t2.x, v[0].y + c1 * t1.y + c2 * t2.y);
        const double2 a2 = make_double2(v[0].x + c2 * t1.x + c1 * t2.x, v[0].y + c2 * t1.y + c1 * t2.y);
        const double2 b1 = cmuli(make_double2(s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y));
        const double2 b2 = cmuli(make_double2(s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y));
        v[0] = cadd(v[0], cadd(t1, t2));
        v[1] = cadd(a1, b1);
        v[2] = cadd(a2, b2);
        v[3] = csub(a2, b2);
        v[4] = csub(a1, b1);
    } else {
        static_assert(P == 8, "radices");
        const double h = 0.70710678118654752440;
        double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft_point(e);
        dft_point(o);
        o[1] = make_double2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));
        o[2] = cmuli(o[2]);
        o[3] = make_double2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = cadd(e[k], o[k]);
            v[k + 4] = csub(e[k], o[k]);
        }
    }
}

// Element i of a line: one slot in nine is left out, so that the strides of
// powers of two of the passes do not meet in the same banks.
__device__ __forceinline__ int fft_slot(int i) { return i + (i >> 3); }
__host__ __device__ constexpr int fft_stride(int n) { return n + (n >> 3) + 1; }

template <int NT, int U, int P>
__device__ __forceinline__ void fft_pass(double2 *S, int nl, int n, int stride, int l, int M,
                                         const double2 *__restrict__ tw, int tmul) {
    constexpr int K = (U + P - 1) / P;  // butterflies per thread: nl n <= U NT
    const int nb = n / P, Mp = M / P, total = nl * nb;
    const float r_nb = 1.0f / (float)nb, r_Mp = 1.0f / (float)Mp;
    double2 v[K][P];
    int dst[K];
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const int b = threadIdx.x + u * NT;
        if (b >= total) continue;
        const int line = div_small(b, r_nb), bb = b - line * nb;
        const int k = div_small(bb, r_Mp), q = bb - k * Mp;
        const double2 *ln = S + line * stride;
#pragma unroll
        for (int j = 0; j < P; ++j) v[u][j] = ln[fft_slot(k * M + q + j * Mp)];
        if (l > 1) {
#pragma unroll
            for (int j = 1; j < P; ++j) v[u][j] = cmul(v[u][j], tw[k * j * Mp * tmul]);
        }
        dst[u] = (line << 16) | (k * Mp + q);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < K; ++u) {
        if ((int)threadIdx.x + u * NT >= total) continue;
        dft_point(v[u]);
        double2 *ln = S + (dst[u] >> 16) * stride;
#pragma unroll
        for (int r = 0; r < P; ++r) ln[fft_slot((dst[u] & 0xffff) + r * l * Mp)] = v[u][r];
    }
    __syncthreads();
}

// Any factor P: each thread forms U outputs, P multiply-adds each.
template <int NT, int U>
__device__ __forceinline__ void fft_pass_any(int P, double2 *S, int nl, int n, int stride, int l, int M,
                                             const double2 *__restrict__ tw, int tmul) {
    const int Mp = M / P;
    const float r_n = 1.0f / (float)n, r_Mp = 1.0f / (float)Mp, r_l = 1.0f / (float)l;
    double2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int o = threadIdx.x + u * NT;
        v[u] = make_double2(0.0, 0.0);
        if (o >= nl * n) continue;
        const int line = div_small(o, r_n), i = o - line * n;
        const int kk = div_small(i, r_Mp), q = i - kk * Mp;
        const int k = kk - div_small(kk, r_l) * l;
        const double2 *ln = S + line * stride;
        const int step = kk * Mp;  // < n
        int t = 0;
        for (int j = 0; j < P; ++j) {
            const double2 a = ln[fft_slot(k * M + q + j * Mp)], w = tw[t * tmul];
            v[u].x += a.x * w.x - a.y * w.y;
            v[u].y += a.x * w.y + a.y * w.x;
            t += step;
            if (t >= n) t -= n;
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int o = threadIdx.x + u * NT;
        if (o >= nl * n) continue;
        const int line = div_small(o, r_n), i = o - line * n;
        S[line * stride + fft_slot(i)] = v[u];
    }
    __syncthreads();
}

// nl lines (line k at S + k fft_stride(n)) of p.n points, nl p.n <= U NT;
// starts behind a barrier and ends with one.  tw[m] = e^{-2 pi i m / (n tmul)}.
template <int NT, int U>
__device__ __forceinline__ void fft_lines(double2 *S, int nl, const FftPlan &p, const double2 *__restrict__ tw) {
    const int n = p.n, stride = fft_stride(n);
    int l = 1, M = n;
    for (int k = 0; k < p.nf; ++k) {
        const int P = p.f[k];
        switch (P) {
        case 8: fft_pass<NT, U, 8>(S, nl, n, stride, l, M, tw, p.tmul); break;
        case 4: fft_pass<NT, U, 4>(S, nl, n, stride, l, M, tw, p.tmul); break;
        case 2: fft_pass<NT, U, 2>(S, nl, n, stride, l, M, tw, p.tmul); break;
        case 3: fft_pass<NT, U, 3>(S, nl, n, stride, l, M, tw, p.tmul); break;
        case 5: fft_pass<NT, U, 5>(S, nl, n, stride, l, M, tw, p.tmul); break;
        default: fft_pass_any<NT, U>(P, S, nl, n, stride, l, M, tw, p.tmul); break;
        }
        l *= P;
        M /= P;
    }
}

}  // namespace lbfss
